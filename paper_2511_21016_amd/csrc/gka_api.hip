// Host side of the C ABI declared in include/gka.h: argument validation, workspace carving and kernel
// launches on the caller's stream. No device allocation and no synchronisation (gka_forward_profile aside); the only
// state kept between calls is the address of gka_forward_static's scratch array on each device.
#include "../../include/gka.h"
#include "gka_kernels.hpp"

#include <mutex>
#include <vector>

namespace {

struct Plan {
    int n_pairs, n_chunks, d;
    bool io_bf16, compute_bf16;
    int64_t stride_b, stride_t, stride_h;
    size_t off_H, off_U, off_hn, off_seg, off_segdecay, off_carry, total;
    int n_segs, seg_len;
    int pairs_per_batch;          // (batch, head) pairs per launch
    int slab_chunks;              // chunks of every pair per launch
    bool recurrent;               // token-by-token kernel: no chunks, no launch plan
    bool wide;                    // d = 256 chunk-wise: the two-phase kernels with float32 operands
    bool pieces;                  // ... which are 16-bit pieces where the tensors and the caller's operands are bf16
    bool small;                   // chunk-wise kernels of the head dimensions 16 and 32 (bf16 tensors and operands)
    bool split;                   // GKA_COMPUTE_BF16_SPLIT (fused kernel only)
    bool fused_shape;             // dtype, operands and head dimension of the fused kernel
    int fused_n_segs, fused_seg_len;
    size_t fused_bytes;           // workspace of the fused kernels alone
};

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr int kStateMinWorkgroups = 512;   // two state-pass workgroups per CU (bf16 operands)
constexpr int kStateMinWorkgroupsF32 = 256;
// Up to this many chunks a state pass is one launch: the second launch that segments need costs as much as walking them
// (d = 64, 5 chunks: 27.8 us per forward pass in two segments, 23.3 us in one; float32, 4 chunks 34.6 and 32.1 us).
constexpr int kStateSingleWalk = 5;
constexpr int kStateMaxWalk = 64;          // chunks a state-pass workgroup walks before segments are added
// Chunk states one launch pair keeps in the workspace unless gka_params::slab_state_bytes says otherwise (tests use
// that to force several slabs on small problems).
constexpr size_t kDefaultSlabStateBytes = (size_t)1 << 30;
using gka::kComputeUnits;                  // the fused kernels run one workgroup on each
// Segments are added up to this many workgroups of the fused kernels (four rounds), or as many as a caller's bound on the
// workspace (gka_params::slab_state_bytes) has room for, one round at least.
constexpr int kFusedMaxWorkgroups = 4 * kComputeUnits;
int fused_max_workgroups(int64_t slab_state_bytes, bool split)
{
    const int64_t fit = slab_state_bytes / (int64_t)gka::fused_workspace_bytes(1, 1, split);
    return slab_state_bytes <= 0 || fit > kFusedMaxWorkgroups ? kFusedMaxWorkgroups : fit < kComputeUnits ? kComputeUnits : (int)fit;
}
// Above this length d = 256 runs chunk-wise. The line is what callers are asked for, not speed: the chunk states need a
// workspace, and calls of up to two chunks have always run without one (sizes queried and allocated once by a program
// would no longer do). Chunk by chunk would be the faster way from 4 to 8 tokens on (us, chunk-wise against token by
// token: 4 pairs, 4 tokens 36 / 55, 16 tokens 36 / 202, 64 tokens 50 / 789, 128 tokens 113 / 1573; 64 pairs, 4 tokens
// 50 / 57, 128 tokens 204 / 1591; 512 pairs, 2 tokens 216 / 110, 4 tokens 213 / 199, 128 tokens 1140 / 5287).
constexpr int kWideMinTokens = 2 * gka::kChunk;
constexpr size_t kMaxPairsPerBatch = 1024;
constexpr size_t kMinSlabChunks = 4;

gka_status check_common(const gka_params *p, bool decode)
{
    if (!p) return GKA_ERR_NULL;
    if (p->B <= 0 || p->H <= 0 || p->n_iter < 0) return GKA_ERR_SHAPE;
    if (!decode && p->T <= 0) return GKA_ERR_SHAPE;
    if (p->d_k <= 0 || p->d_v <= 0) return GKA_ERR_SHAPE;
    if (p->phase < GKA_PHASE_ALL || p->phase > GKA_PHASE_SOLVE) return GKA_ERR_UNSUPPORTED;
    if (p->d_k != p->d_v) return GKA_ERR_UNSUPPORTED;
    if (p->d_k != 16 && p->d_k != 32 && p->d_k != 64 && p->d_k != 128 && p->d_k != 256) return GKA_ERR_UNSUPPORTED;
    if (p->io_dtype != GKA_F32 && p->io_dtype != GKA_BF16) return GKA_ERR_UNSUPPORTED;
    if (p->compute < GKA_COMPUTE_F32 || p->compute > GKA_COMPUTE_BF16_SPLIT) return GKA_ERR_UNSUPPORTED;
    if (p->io_dtype == GKA_F32 && p->compute != GKA_COMPUTE_F32) return GKA_ERR_UNSUPPORTED;
    if (!decode && p->chunk != gka::kChunk) return GKA_ERR_UNSUPPORTED;
    if ((int64_t)p->B * p->H > (int64_t)1 << 24) return GKA_ERR_SHAPE;
    if (!(p->lambda_scale >= 0.0f)) return GKA_ERR_SHAPE;
    if (p->state_layout != GKA_STATE_FULL && p->state_layout != GKA_STATE_H_LOWER_BLOCKS) return GKA_ERR_UNSUPPORTED;
    if (p->slab_state_bytes < 0 || p->walk_chunks < 0) return GKA_ERR_SHAPE;
    if (p->state_layout == GKA_STATE_H_LOWER_BLOCKS && p->d_k == 256) return GKA_ERR_UNSUPPORTED;
    if (p->path < GKA_PATH_AUTO || p->path > GKA_PATH_RECURRENT) return GKA_ERR_UNSUPPORTED;
    return GKA_OK;
}

// head dimensions of the chunk-wise kernels (the others run token by token)
bool chunked_dim(int d) { return d == 64 || d == 128; }

// Chunks per segment of the fused kernels: the number of segments whose estimated time is the shortest. A launch runs in
// ceil(workgroups / 256) rounds; a workgroup's walk costs kStart, then kIter + kPass per pass for an iteration (two chunks;
// split operands: one), and kScan for each earlier segment whose summary its start state is composed of; the summary launch
// walks every segment but the last once more (constants in us, from launches of 4 to 384 pairs). Measured against the former
// rule, as few segments as give every CU a workgroup, us per forward pass: 16 pairs x 1337 tokens 66.2 -> 49.2, 36 x 2000
// 131 -> 103 (288 workgroups -> 216), 48 x 3000 234 -> 173, 80 x 4096 464 -> 382, 100 x 4096 597 -> 497, 300 x 4096 1697 -> 1426,
// 200 x 4096 944 -> 875; split operands, 12 passes, 48 x 2600 471 -> 352; 64 x 4096 and 32 x 32768 keep their segments.
int fused_segment(int n_pairs, int n_chunks, int n_iter, bool split, int max_workgroups)
{
    constexpr float kStart = 10.0f, kScan = 1.3f, kSummaryStart = 5.0f, kSummaryChunk = 2.1f;
    const float iteration = split ? 15.0f + 1.6f * n_iter : 13.5f + 1.15f * n_iter;
    const int step = split ? 1 : 2;
    const auto rounds = [](int64_t workgroups) { return (float)((workgroups + kComputeUnits - 1) / kComputeUnits); };
    int best = n_chunks, last = 0;
    float best_us = 0.0f;
    for (int64_t segs = 1; segs <= (n_chunks + step - 1) / step; ++segs) {
        int len = (int)((n_chunks + segs - 1) / segs);
        len += len % step;
        if (len == last) continue;
        last = len;
        const int64_t n = (n_chunks + len - 1) / len;
        if (n > 1 && n * n_pairs > max_workgroups) break;
        float us = rounds(n * n_pairs) * (kStart + iteration * (len / step) + kScan * (n - 1));
        if (n > 1) us += kSummaryStart + rounds((n - 1) * n_pairs) * kSummaryChunk * len;
        if (segs == 1 || us < best_us) {
            best = len;
            best_us = us;
        }
    }
    return best;
}

// most_workgroups: of the fused kernels, where their scratch has a fixed size (0: the library's choice); fused_bytes is then what
// this plan takes.
gka_status make_plan(const gka_params *p, Plan *pl, bool readout_only = false, int most_workgroups = 0)
{
    gka_status s = check_common(p, false);
    if (s != GKA_OK) return s;
    pl->d = p->d_k;
    pl->n_pairs = p->B * p->H;
    pl->n_chunks = (p->T + gka::kChunk - 1) / gka::kChunk;
    pl->io_bf16 = p->io_dtype == GKA_BF16;
    pl->compute_bf16 = p->compute != GKA_COMPUTE_F32;
    pl->split = p->compute == GKA_COMPUTE_BF16_SPLIT;
    // d = 16, 32: chunk-wise kernels of their own for bf16 tensors with bf16 operands (what GKA_PATH_AUTO and
    // GKA_PATH_TWO_PHASE select there), else token by token
    pl->small = pl->d <= 32 && pl->io_bf16 && p->compute == GKA_COMPUTE_BF16 && !readout_only &&
                (p->path == GKA_PATH_AUTO || p->path == GKA_PATH_TWO_PHASE);
    // d = 256: GKA_PATH_AUTO takes the chunk-wise kernels with float32 operands (the token-by-token kernel's arithmetic)
    // above kWideMinTokens
    pl->wide = pl->d == 256 && p->path == GKA_PATH_AUTO && p->T > kWideMinTokens && !pl->split && !readout_only;
    pl->pieces = pl->wide && pl->io_bf16 && p->compute == GKA_COMPUTE_BF16;
    pl->recurrent = !pl->small && !pl->wide && (p->path == GKA_PATH_RECURRENT || !chunked_dim(pl->d));
    if (pl->recurrent && (p->path == GKA_PATH_TWO_PHASE || p->path == GKA_PATH_FUSED || readout_only))
        return GKA_ERR_UNSUPPORTED;
    if ((int64_t)pl->n_pairs * pl->n_chunks > (int64_t)0x7fffffff) return GKA_ERR_SHAPE;
    if (p->stride_b == 0 && p->stride_t == 0 && p->stride_h == 0) {
        pl->stride_h = p->d_k;
        pl->stride_t = (int64_t)p->H * p->d_k;
        pl->stride_b = (int64_t)p->T * p->H * p->d_k;
    } else {
        if (p->stride_b <= 0 || p->stride_t <= 0 || p->stride_h <= 0) return GKA_ERR_SHAPE;
        if (p->stride_h < p->d_k && p->H > 1) return GKA_ERR_SHAPE;
        if (p->stride_t % 4 || p->stride_h % 4 || p->stride_b % 4) return GKA_ERR_SHAPE;  // vector stores
        // bf16 operands: k rows are copied 16 bytes at a time, addressed with 32-bit byte offsets within a chunk
        if (pl->compute_bf16 && (p->stride_t % 8 || p->stride_h % 8 || p->stride_b % 8)) return GKA_ERR_SHAPE;
        if (pl->compute_bf16 && p->stride_t >= (1 << 23)) return GKA_ERR_UNSUPPORTED;
        pl->stride_b = p->stride_b;
        pl->stride_t = p->stride_t;
        pl->stride_h = p->stride_h;
    }
    if (pl->wide) pl->compute_bf16 = false;
    if (pl->small) {
        if ((int64_t)pl->n_pairs * pl->n_chunks > (int64_t)0x7fffffff / 4) return GKA_ERR_SHAPE;
        pl->fused_shape = false;
        pl->fused_bytes = 0;
        pl->total = align_up(gka::small_dim_workspace_bytes(pl->n_pairs, pl->n_chunks, pl->d, true), 256);
        return GKA_OK;
    }
    if (pl->recurrent) {
        // states stay in registers; only d = 256 streams U through memory and needs room for it when the caller does
        // not ask for U_final
        pl->fused_shape = false;
        pl->fused_bytes = 0;
        pl->total = 256 + (pl->d == 256 ? align_up((size_t)pl->n_pairs * pl->d * pl->d * sizeof(float), 256) : 0);
        return GKA_OK;
    }
    // The work is cut into launches of (a batch of pairs) x (a slab of consecutive chunks), slabs in sequence order,
    // so that the chunk states one launch pair writes and reads (state pass, then solve) fit a bounded workspace,
    // which every launch pair reuses; the running states are carried between slabs in fp32. (Slabs small enough to
    // stay in the last-level cache were measured slower than one launch pair: more launches, shorter walks.)
    const size_t per_chunk = gka::ws_H_bytes_per_chunk(pl->d, pl->compute_bf16) +
                             gka::ws_U_bytes_per_chunk(pl->d, pl->compute_bf16);
    size_t ppb = pl->n_pairs < kMaxPairsPerBatch ? pl->n_pairs : kMaxPairsPerBatch;
    const size_t budget = p->slab_state_bytes > 0 ? (size_t)p->slab_state_bytes : kDefaultSlabStateBytes;
    if (pl->wide) {
        // (512 KiB per chunk: kMinSlabChunks of 1024 pairs would take twice the budget)
        const size_t least = (size_t)pl->n_chunks < kMinSlabChunks ? (size_t)pl->n_chunks : kMinSlabChunks;
        const size_t fit = budget / (least * per_chunk);
        if (ppb > fit) ppb = fit > 0 ? fit : 1;
    }
    size_t slab = budget / (ppb * per_chunk);
    if (slab < kMinSlabChunks) slab = kMinSlabChunks;
    if (slab > (size_t)pl->n_chunks) slab = pl->n_chunks;
    pl->pairs_per_batch = (int)ppb;
    pl->slab_chunks = (int)slab;
    const size_t nc = ppb * slab;
    pl->off_H = 0;
    pl->off_U = align_up(pl->off_H + nc * gka::ws_H_bytes_per_chunk(pl->d, pl->compute_bf16), 256);
    pl->off_hn = align_up(pl->off_U + nc * gka::ws_U_bytes_per_chunk(pl->d, pl->compute_bf16), 256);
    pl->off_seg = align_up(pl->off_hn + nc * gka::ws_hn_bytes_per_chunk(pl->d), 256);
    // Segments of the chunk scan. A workgroup walks its chunks one after the other (a few microseconds each), and a
    // segmented pass reads k and v twice, so: one segment unless that leaves CUs idle or makes the walk longer than
    // about 64 chunks; never fewer than two chunks per segment.
    // (a plain readout walks U only: half the workgroups of a segment have nothing to do)
    int wg_per_seg = gka::state_pass_workgroups_per_segment(pl->pairs_per_batch, pl->d, pl->compute_bf16);
    if (readout_only && wg_per_seg > 1) wg_per_seg /= 2;
    int n_segs = ((pl->compute_bf16 ? kStateMinWorkgroups : kStateMinWorkgroupsF32) + wg_per_seg - 1) / wg_per_seg;
    if (pl->slab_chunks <= kStateSingleWalk) n_segs = 1;
    if (n_segs < pl->slab_chunks / kStateMaxWalk) n_segs = pl->slab_chunks / kStateMaxWalk;
    if (n_segs > pl->slab_chunks / 2) n_segs = pl->slab_chunks / 2;
    if (n_segs < 1) n_segs = 1;
    pl->seg_len = (pl->slab_chunks + n_segs - 1) / n_segs;
    pl->n_segs = (pl->slab_chunks + pl->seg_len - 1) / pl->seg_len;
    // (one segment needs no summaries, one slab carries nothing)
    const size_t n_summaries = pl->n_segs > 1 ? (size_t)pl->pairs_per_batch * pl->n_segs : 0;
    pl->off_segdecay = align_up(pl->off_seg + n_summaries * 2 * pl->d * pl->d * sizeof(float), 256);
    pl->off_carry = align_up(pl->off_segdecay + n_summaries * sizeof(float), 256);
    // two ping-pong pairs of fp32 (H, U) carried from slab to slab
    const size_t n_carried = pl->slab_chunks < pl->n_chunks ? (size_t)4 * pl->pairs_per_batch : 0;
    pl->total = align_up(pl->off_carry + n_carried * pl->d * pl->d * sizeof(float), 256);
    // Fused kernel: one workgroup per (pair, segment of the chunk walk); an even number of chunks per segment, because a
    // workgroup takes its chunks two at a time.
    pl->fused_shape = pl->io_bf16 && pl->compute_bf16 && pl->d == 128 && !readout_only;
    pl->fused_bytes = 0;
    if (pl->fused_shape) {
        int seg_len;
        int max_workgroups = fused_max_workgroups(p->slab_state_bytes, pl->split);
        if (most_workgroups > 0 && max_workgroups > most_workgroups) max_workgroups = most_workgroups;
        if (p->walk_chunks > 0) {
            seg_len = p->walk_chunks < pl->n_chunks ? p->walk_chunks : pl->n_chunks;
        } else {
            seg_len = fused_segment(pl->n_pairs, pl->n_chunks, p->n_iter, pl->split, max_workgroups);
        }
        if (!pl->split) seg_len += seg_len & 1;
        pl->fused_seg_len = seg_len;
        pl->fused_n_segs = (pl->n_chunks + seg_len - 1) / seg_len;
        if ((int64_t)pl->n_pairs * pl->fused_n_segs > (int64_t)0x7fffffff) return GKA_ERR_SHAPE;
        // The size asked for does not shrink with the number of pairs or tokens or depend on the number of passes, as the
        // segments may: a workspace serves every smaller call.
        int64_t workgroups = (int64_t)pl->n_pairs * pl->fused_n_segs;
        if (p->walk_chunks == 0 && most_workgroups == 0) {
            const int64_t finest = (int64_t)pl->n_pairs * (pl->split ? pl->n_chunks : (pl->n_chunks + 1) / 2);
            workgroups = finest < max_workgroups ? finest : max_workgroups;
            if (workgroups < pl->n_pairs) workgroups = pl->n_pairs;
        }
        pl->fused_bytes = align_up(gka::fused_workspace_bytes((int)workgroups, 1, pl->split), 256);
        // (a caller that insists on the fused kernels needs no room for the two-phase kernels' chunk states)
        if (p->path == GKA_PATH_FUSED || pl->split || pl->fused_bytes > pl->total) pl->total = pl->fused_bytes;
    }
    return GKA_OK;
}

}  // namespace

extern "C" {

size_t gka_forward_workspace_bytes(const gka_params *p)
{
    Plan pl;
    if (make_plan(p, &pl) != GKA_OK) return 0;
    return pl.total;
}

}  // extern "C"

namespace {

// Events around the two phases of every batch (profiling entry point only).
struct PhaseEvents {
    std::vector<hipEvent_t> ev;
    bool ok = true;
    void mark(hipStream_t stream)
    {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) { ok = false; return; }
        if (hipEventRecord(e, stream) != hipSuccess) ok = false;
        ev.push_back(e);
    }
    ~PhaseEvents()
    {
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
    }
};

// A second right-hand side (value + remainder) for the systems of a solve, and where its and the first one's results go
// besides p->xhat_out.
struct SecondRhs {
    const void *q, *q_lo;
    float *xhat;
    void *first_hi, *first_lo, *hi;          // bf16: value and remainder of the first result, value of the second
};

// The final states replace the initial ones in the caller's buffers.
bool states_in_place(const float *H_init, const float *U_init, const float *H_final, const float *U_final)
{
    return H_final && (H_final == H_init || U_final == U_init);
}

gka_status forward_impl(const gka_params *p, const void *q, const void *k, const void *v, const float *gate,
                        const float *lambda, void *o, const float *H_init, const float *U_init, float *H_final,
                        float *U_final, float *fro_out, void *workspace, size_t workspace_bytes,
                        void *hip_stream, PhaseEvents *prof, bool readout_only = false, bool solve_only = false,
                        const SecondRhs *second = nullptr, int most_workgroups = 0)
{
    Plan pl;
    gka_status s = make_plan(p, &pl, readout_only, most_workgroups);
    if (s != GKA_OK) return s;
    if (!q || !k || !v || !gate || !o) return GKA_ERR_NULL;
    if (!lambda && !(p->lambda_scale > 0.0f)) return GKA_ERR_NULL;      // neither lambda_t nor the rule for it
    if ((H_init == nullptr) != (U_init == nullptr)) return GKA_ERR_NULL;
    if ((H_final == nullptr) != (U_final == nullptr)) return GKA_ERR_NULL;
    if (!workspace || workspace_bytes < pl.total || ((uintptr_t)workspace & 255)) return GKA_ERR_WORKSPACE;
    hipStream_t stream = (hipStream_t)hip_stream;
    char *ws = (char *)workspace;

    if (pl.small) {
        if (p->phase != GKA_PHASE_ALL || solve_only) return GKA_ERR_UNSUPPORTED;
        gka::SmallArgs sm = {};
        sm.q = q; sm.k = k; sm.v = v; sm.o = o;
        sm.stride_b = pl.stride_b; sm.stride_t = pl.stride_t; sm.stride_h = pl.stride_h;
        sm.d = pl.d;
        sm.gate = gate; sm.lambda = lambda; sm.beta = p->beta; sm.alpha = p->alpha; sm.lambda_scale = p->lambda_scale;
        sm.xhat_out = p->xhat_out; sm.xhat_row = pl.d; sm.xhat_zero_upper = false;
        sm.fro_out = fro_out;
        sm.H_init = H_init; sm.U_init = U_init; sm.H_final = H_final; sm.U_final = U_final;
        sm.T = p->T; sm.H = p->H; sm.n_pairs = pl.n_pairs; sm.n_chunks = pl.n_chunks; sm.n_iter = p->n_iter;
        // (profiling: all of it is reported as the solve phase)
        if (prof) { prof->mark(stream); prof->mark(stream); }
        if (gka::launch_small_dim_forward(sm, ws, stream) != hipSuccess) return GKA_ERR_LAUNCH;
        if (prof) prof->mark(stream);
        return GKA_OK;
    }
    if (pl.recurrent) {
        if (p->phase != GKA_PHASE_ALL || pl.split || solve_only) return GKA_ERR_UNSUPPORTED;
        gka::DecodeArgs da = {};
        da.H_in = H_init; da.U_in = U_init;
        da.H_state = H_final;
        da.U_state = U_final ? U_final : (pl.d == 256 ? (float *)(ws + 256) : nullptr);
        da.h_out_full = true;
        da.h_lower_blocks = p->state_layout == GKA_STATE_H_LOWER_BLOCKS && chunked_dim(pl.d);
        da.q = q; da.k = k; da.v = v; da.gate = gate; da.lambda = lambda; da.o = o;
        da.stride_b = pl.stride_b; da.stride_t = pl.stride_t; da.stride_h = pl.stride_h;
        da.beta = p->beta; da.alpha = p->alpha; da.lambda_scale = p->lambda_scale;
        da.fro_out = fro_out; da.xhat_out = p->xhat_out;
        da.n_iter = p->n_iter; da.T = p->T; da.H = p->H;
        // (profiling: all of it is reported as the solve phase)
        if (prof) { prof->mark(stream); prof->mark(stream); }
        if (gka::launch_decode_step(da, pl.n_pairs, pl.d, pl.io_bf16, stream) != hipSuccess) return GKA_ERR_LAUNCH;
        if (prof) prof->mark(stream);
        return GKA_OK;
    }
    const bool fused_ok = pl.fused_shape && !p->xhat_out && !solve_only && p->phase == GKA_PHASE_ALL;
    if ((p->path == GKA_PATH_FUSED || pl.split) && !fused_ok) return GKA_ERR_UNSUPPORTED;
    if (pl.wide && p->phase != GKA_PHASE_ALL) return GKA_ERR_UNSUPPORTED;
    if (pl.split && p->path == GKA_PATH_TWO_PHASE) return GKA_ERR_UNSUPPORTED;     // only the fused kernel splits
    if (fused_ok && p->path != GKA_PATH_TWO_PHASE) {
        gka::FusedArgs fa = {};
        fa.q = q; fa.k = k; fa.v = v; fa.gate = gate; fa.lambda = lambda; fa.o = o; fa.fro_out = fro_out;
        fa.beta = p->beta; fa.alpha = p->alpha; fa.lambda_scale = p->lambda_scale;
        fa.H_init = H_init; fa.U_init = U_init; fa.H_final = H_final; fa.U_final = U_final;
        fa.h_init_lower_blocks = p->state_layout == GKA_STATE_H_LOWER_BLOCKS;
        fa.stride_b = pl.stride_b; fa.stride_t = pl.stride_t; fa.stride_h = pl.stride_h;
        fa.H = p->H; fa.T = p->T; fa.n_iter = p->n_iter;
        fa.n_pairs = pl.n_pairs; fa.n_chunks = pl.n_chunks;
        fa.n_segs = pl.fused_n_segs; fa.seg_len = pl.fused_seg_len;
        fa.seg_buf = nullptr; fa.seg_logdecay = nullptr;
        // (profiling: the summary launch is reported as the state phase, the chunk walk as the solve phase)
        if (prof) prof->mark(stream);
        if (gka::launch_fused_forward(fa, ws, stream, 1, pl.split) != hipSuccess) return GKA_ERR_LAUNCH;
        if (prof) prof->mark(stream);
        if (gka::launch_fused_forward(fa, ws, stream, 2, pl.split) != hipSuccess) return GKA_ERR_LAUNCH;
        if (prof) prof->mark(stream);
        return GKA_OK;
    }

    gka::StatePassArgs sa = {};
    sa.k = k; sa.v = v; sa.gate = gate; sa.beta = p->beta;
    sa.H_init = H_init; sa.U_init = U_init;
    sa.H_final = H_final; sa.U_final = U_final;
    sa.ws_H = ws + pl.off_H; sa.ws_U = ws + pl.off_U; sa.ws_hn = (float *)(ws + pl.off_hn);
    sa.stride_b = pl.stride_b; sa.stride_t = pl.stride_t; sa.stride_h = pl.stride_h;
    sa.H = p->H; sa.T = p->T;
    sa.n_segs = pl.n_segs; sa.seg_len = pl.seg_len;
    sa.seg_buf = (float *)(ws + pl.off_seg); sa.seg_logdecay = (float *)(ws + pl.off_segdecay);
    sa.init_mode = 0; sa.final_mode = 0; sa.write_frags = 1;
    gka::SolveArgs so = {};
    so.q = q; so.k = k; so.v = v; so.gate = gate; so.lambda = lambda; so.o = o; so.fro_out = fro_out;
    if (second) {
        so.q2 = second->q; so.q2_lo = second->q_lo; so.xhat2_out = second->xhat;
        so.xhat_hi = second->first_hi; so.xhat_lo = second->first_lo; so.xhat2_hi = second->hi;
    }
    so.beta = p->beta; so.alpha = p->alpha; so.lambda_scale = p->lambda_scale;
    so.xhat_out = p->xhat_out;
    // plain readout y_t = U_t q_t (used by the backward pass): needs alpha = 0 from the caller; no H states, no solve
    sa.only_u = readout_only; so.readout_only = readout_only;
    // the solve alone (latent sketching): needs xhat_out; no U states, no readout, o is left untouched
    sa.only_h = solve_only; so.solve_only = solve_only;
    so.ws_H = sa.ws_H; so.ws_U = sa.ws_U; so.ws_hn = sa.ws_hn;
    so.stride_b = pl.stride_b; so.stride_t = pl.stride_t; so.stride_h = pl.stride_h;
    so.H = p->H; so.T = p->T; so.n_iter = p->n_iter;
    so.init_states = H_init != nullptr;
    sa.pieces = so.pieces = pl.pieces;
    // d = 256 with the final states in the buffers of the initial ones: one segment, whose workgroups read the part of a state
    // that they write. (With several segments the last one's workgroups would write what the others may not have read yet;
    // several slabs read and write them in different launches.)
    if (pl.wide && states_in_place(H_init, U_init, H_final, U_final) && pl.slab_chunks >= pl.n_chunks) sa.n_segs = 1;
    const bool one_launch = pl.pairs_per_batch >= pl.n_pairs && pl.slab_chunks >= pl.n_chunks;
    // With a single phase requested the workspace must cover the whole problem.
    if (p->phase != GKA_PHASE_ALL && !one_launch) return GKA_ERR_UNSUPPORTED;
    const size_t state_elems = (size_t)pl.pairs_per_batch * pl.d * pl.d;
    float *carry = (float *)(ws + pl.off_carry);               // [2][2][pairs_per_batch, d, d]
    for (int pair0 = 0; pair0 < pl.n_pairs; pair0 += pl.pairs_per_batch) {
        const int np = pl.n_pairs - pair0 < pl.pairs_per_batch ? pl.n_pairs - pair0 : pl.pairs_per_batch;
        int slab_index = 0;
        for (int chunk0 = 0; chunk0 < pl.n_chunks; chunk0 += pl.slab_chunks, ++slab_index) {
            const int nch = pl.n_chunks - chunk0 < pl.slab_chunks ? pl.n_chunks - chunk0 : pl.slab_chunks;
            const bool first = chunk0 == 0, last = chunk0 + nch >= pl.n_chunks;
            sa.pair0 = so.pair0 = pair0;
            sa.chunk0 = so.chunk0 = chunk0;
            sa.n_chunks = so.n_chunks = nch;
            // states enter from the caller (first slab) or from the previous slab, and leave to the next slab or to
            // the caller (last slab)
            float *in = carry + (size_t)((slab_index + 1) & 1) * 2 * state_elems;
            float *out = carry + (size_t)(slab_index & 1) * 2 * state_elems;
            sa.H_init = first ? H_init : in;
            sa.U_init = first ? U_init : in + state_elems;
            sa.init_pair0 = first ? pair0 : 0;
            // states carried between slabs are always complete
            sa.h_init_lower_blocks = first && p->state_layout == GKA_STATE_H_LOWER_BLOCKS;
            sa.H_final = last ? H_final : out;
            sa.U_final = last ? U_final : out + state_elems;
            sa.final_pair0 = last ? pair0 : 0;
            if (prof) prof->mark(stream);
            if (p->phase != GKA_PHASE_SOLVE &&
                gka::launch_state_pass(sa, np, pl.d, pl.io_bf16, pl.compute_bf16, stream) != hipSuccess)
                return GKA_ERR_LAUNCH;
            if (prof) prof->mark(stream);
            if (p->phase != GKA_PHASE_STATES &&
                gka::launch_chunk_solve(so, np, pl.d, pl.io_bf16, pl.compute_bf16, stream) != hipSuccess)
                return GKA_ERR_LAUNCH;
            if (prof) prof->mark(stream);
        }
    }
    return GKA_OK;
}

}  // namespace

extern "C" {

gka_status gka_forward(const gka_params *p, const void *q, const void *k, const void *v, const float *gate,
                       const float *lambda, void *o, const float *H_init, const float *U_init, float *H_final,
                       float *U_final, float *fro_out, void *workspace, size_t workspace_bytes,
                       void *hip_stream)
{
    return forward_impl(p, q, k, v, gate, lambda, o, H_init, U_init, H_final, U_final, fro_out, workspace,
                        workspace_bytes, hip_stream, nullptr);
}

gka_status gka_forward_profile(const gka_params *p, const void *q, const void *k, const void *v, const float *gate,
                               const float *lambda, void *o, const float *H_init, const float *U_init,
                               float *H_final, float *U_final, float *fro_out, void *workspace,
                               size_t workspace_bytes, void *hip_stream, float *ms_states, float *ms_solve,
                               int32_t *n_solve_launches)
{
    if (!ms_states || !ms_solve || !n_solve_launches) return GKA_ERR_NULL;
    PhaseEvents prof;
    gka_status s = forward_impl(p, q, k, v, gate, lambda, o, H_init, U_init, H_final, U_final, fro_out, workspace,
                                workspace_bytes, hip_stream, &prof);
    if (s != GKA_OK) return s;
    if (!prof.ok || prof.ev.empty() || hipEventSynchronize(prof.ev.back()) != hipSuccess) return GKA_ERR_LAUNCH;
    float t_states = 0.0f, t_solve = 0.0f;
    for (size_t i = 0; i + 2 < prof.ev.size(); i += 3) {
        float a = 0.0f, b = 0.0f;
        if (hipEventElapsedTime(&a, prof.ev[i], prof.ev[i + 1]) != hipSuccess) return GKA_ERR_LAUNCH;
        if (hipEventElapsedTime(&b, prof.ev[i + 1], prof.ev[i + 2]) != hipSuccess) return GKA_ERR_LAUNCH;
        t_states += a;
        t_solve += b;
    }
    *ms_states = t_states;
    *ms_solve = t_solve;
    *n_solve_launches = (int32_t)(prof.ev.size() / 3);
    return GKA_OK;
}

// ---- gka_forward_static: the fused kernels with their scratch in a fixed device array --------------------------
namespace {
// Segment summaries and parked states of the fused kernels: GKA_STATIC_SCRATCH_BYTES of summaries and parked U for as many
// workgroups as they hold, and room for the H that each of them parks beside U with split operands. Every GPU the library runs
// on holds its own copy until the process ends. In host code the array's name is only a handle: its device address comes from
// hipGetSymbolAddress, once per device, and is what kernels and copies are given.
constexpr size_t kStateBytes = 128 * 128 * sizeof(float);
constexpr int kStaticWorkgroups = GKA_STATIC_SCRATCH_BYTES / (3 * kStateBytes + sizeof(float));
constexpr size_t kStaticBytes = GKA_STATIC_SCRATCH_BYTES + kStaticWorkgroups * kStateBytes;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};

gka_status static_scratch(void **ptr)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GKA_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GKA_ERR_LAUNCH;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return GKA_OK;
}
}  // namespace

gka_status gka_forward_static(const gka_params *p, const void *q, const void *k, const void *v, const float *gate,
                              const float *lambda, void *o, const float *H_init, const float *U_init, float *H_final,
                              float *U_final, float *fro_out, void *hip_stream)
{
    Plan pl;
    gka_status s = make_plan(p, &pl, false, kStaticWorkgroups);
    if (s != GKA_OK) return s;
    if (!pl.fused_shape || p->path == GKA_PATH_TWO_PHASE) return GKA_ERR_UNSUPPORTED;
    if ((int64_t)pl.n_pairs * pl.fused_n_segs > kStaticWorkgroups) return GKA_ERR_STATIC_SCRATCH;
    void *ws = nullptr;
    s = static_scratch(&ws);
    if (s != GKA_OK) return s;
    gka_params pf = *p;
    pf.path = GKA_PATH_FUSED;            // (anything the fused kernels do not cover: GKA_ERR_UNSUPPORTED)
    return forward_impl(&pf, q, k, v, gate, lambda, o, H_init, U_init, H_final, U_final, fro_out, ws, kStaticBytes, hip_stream,
                        nullptr, false, false, nullptr, kStaticWorkgroups);
}

namespace {
gka_status decode_impl(const gka_params *p, int n_tokens, float *H_state, float *U_state, const void *q, const void *k,
                       const void *v, const float *gate, const float *lambda, void *o, void *hip_stream)
{
    gka_status s = check_common(p, true);
    if (s != GKA_OK) return s;
    if (n_tokens <= 0) return GKA_ERR_SHAPE;
    if (!H_state || !U_state || !q || !k || !v || !gate || !o) return GKA_ERR_NULL;
    if (!lambda && !(p->lambda_scale > 0.0f)) return GKA_ERR_NULL;
    gka::DecodeArgs da = {};
    da.H_in = H_state; da.U_in = U_state;
    da.H_state = H_state; da.U_state = U_state;
    da.q = q; da.k = k; da.v = v; da.gate = gate; da.lambda = lambda; da.o = o;
    da.stride_h = p->d_k; da.stride_t = (int64_t)p->H * p->d_k; da.stride_b = (int64_t)n_tokens * p->H * p->d_k;
    da.beta = p->beta; da.alpha = p->alpha; da.lambda_scale = p->lambda_scale;
    da.n_iter = p->n_iter;
    da.T = n_tokens; da.H = p->H;
    da.h_lower_blocks = p->state_layout == GKA_STATE_H_LOWER_BLOCKS && chunked_dim(p->d_k);
    if (gka::launch_decode_step(da, p->B * p->H, p->d_k, p->io_dtype == GKA_BF16, (hipStream_t)hip_stream) !=
        hipSuccess)
        return GKA_ERR_LAUNCH;
    return GKA_OK;
}
}  // namespace

gka_status gka_decode_step(const gka_params *p, float *H_state, float *U_state, const void *q, const void *k,
                           const void *v, const float *gate, const float *lambda, void *o, void *hip_stream)
{
    return decode_impl(p, 1, H_state, U_state, q, k, v, gate, lambda, o, hip_stream);
}

gka_status gka_decode_tokens(const gka_params *p, float *H_state, float *U_state, const void *q, const void *k,
                             const void *v, const float *gate, const float *lambda, void *o, void *hip_stream)
{
    if (!p) return GKA_ERR_NULL;
    if (p->stride_b != 0 || p->stride_t != 0 || p->stride_h != 0) return GKA_ERR_UNSUPPORTED;
    return decode_impl(p, p->T, H_state, U_state, q, k, v, gate, lambda, o, hip_stream);
}

namespace {
// Segments of the fused readout's chunk scan: two workgroups per CU when the pairs alone do not give that many,
// never fewer than two chunks per segment.
constexpr int kReadoutMinWorkgroups = 512;
void plan_readout_segments(int n_pairs, int n_chunks, int *n_segs, int *seg_len)
{
    int ns = (kReadoutMinWorkgroups + n_pairs - 1) / n_pairs;
    if (ns > n_chunks / 2) ns = n_chunks / 2;
    if (ns < 1) ns = 1;
    *seg_len = (n_chunks + ns - 1) / ns;
    *n_segs = (n_chunks + *seg_len - 1) / *seg_len;
}

// ... of the reverse recurrences' walk: one workgroup per CU
constexpr int kReverseMinWorkgroups = 256;
void plan_reverse_segments(int n_pairs, int n_chunks, int *n_segs, int *seg_len)
{
    int ns = (kReverseMinWorkgroups + n_pairs - 1) / n_pairs;
    if (ns > n_chunks / 2) ns = n_chunks / 2;
    if (ns < 1) ns = 1;
    *seg_len = (n_chunks + ns - 1) / ns;
    *n_segs = (n_chunks + *seg_len - 1) / *seg_len;
}

// Segments of the two solves' walk (gka_fused.hip) and the finer parts of them whose summaries are formed: the readouts, which
// start from the same summaries, walk a part each. seg_len is a multiple of sum_len and even.
struct WalkSegments {
    int seg_len, n_segs, sum_len, n_sums;
};
// Most summaries and most segments of all pairs together, whatever the number of passes: what the workspace has room for. A part
// of a segment has two chunks at least.
struct WalkRoom {
    int64_t sums, segs;
};
WalkRoom walk_room(int n_pairs, int n_chunks, int walk_chunks)
{
    const int64_t finest = (int64_t)n_pairs * ((n_chunks + 1) / 2);
    if (walk_chunks > 0) return {finest, finest};
    const int64_t segs = n_pairs > kFusedMaxWorkgroups ? n_pairs : kFusedMaxWorkgroups;
    const int64_t sums = (int64_t)kFusedMaxWorkgroups + n_pairs;
    return {finest < sums ? finest : sums, finest < segs ? finest : segs};
}
WalkSegments plan_walk_segments(int n_pairs, int n_chunks, int n_iter, int walk_chunks)
{
    int rs_n, rs_len;
    plan_readout_segments(n_pairs, n_chunks, &rs_n, &rs_len);
    int len = walk_chunks <= 0 ? fused_segment(n_pairs, n_chunks, 2 * n_iter, false, kFusedMaxWorkgroups)
                               : walk_chunks < n_chunks ? walk_chunks : n_chunks;
    // (a segment of more chunks than there are has no more parts for it)
    int parts = ((len < n_chunks ? len : n_chunks) + rs_len - 1) / rs_len;
    len += len & 1;
    if (parts > len / 2) parts = len / 2;            // (two chunks at least)
    const WalkRoom room = walk_room(n_pairs, n_chunks, walk_chunks);
    for (;; --parts) {                               // (with one part a summary is a segment, for which there is room)
        WalkSegments s;
        s.sum_len = (len + parts - 1) / parts;
        if (s.sum_len * parts % 2) ++s.sum_len;
        s.seg_len = s.sum_len * parts;
        s.n_segs = (n_chunks + s.seg_len - 1) / s.seg_len;
        s.n_sums = (n_chunks + s.sum_len - 1) / s.sum_len;
        if (parts == 1 || (int64_t)n_pairs * s.n_sums <= room.sums) return s;
    }
}

// Tensors of the backward pass in the tensors' dtype: those of float32 tensors alone, those of both, those of bf16 tensors.
enum { IO_Y, IO_DXT, IO_HX, IO_KR, IO_VR, IO_DYR, IO_XR, IO_XTR, IO_R1, IO_R2, IO_R3, IO_R4,
       IO_RHS, IO_BF16_FIRST = IO_RHS, IO_X, IO_XT, IO_PR, IO_SCRATCH, IO_HK, IO_VPR, IO_R5,
       IO_RHS_LO, IO_REMAINDERS = IO_RHS_LO, IO_X_LO, IO_XT_LO, IO_TENSORS };

struct BackwardPlan {
    size_t n_elems, n_tokens, esz;
    size_t off_f32[3];        // xhat, p; bf16 tensors: U^T dy
    size_t off_io[IO_TENSORS];
    size_t off_m[9];          // gate_rev, zeros, s, fro, c, C, p . H x, k . dk / beta, v . dv / beta
    size_t off_fin[3];        // final states of three reverse readouts (gradients at the initial states)
    size_t off_fwd, fwd_bytes, total;
    bool strided;             // q, k, v, dy come with explicit strides
    size_t off_pack[4];       // their packed copies
};
gka_status make_backward_plan(const gka_params *p, BackwardPlan *bp)
{
    gka_status s = check_common(p, false);
    if (s != GKA_OK) return s;
    if (!chunked_dim(p->d_k) || p->path == GKA_PATH_RECURRENT) return GKA_ERR_UNSUPPORTED;
    if (p->phase != GKA_PHASE_ALL || p->compute == GKA_COMPUTE_BF16_SPLIT) return GKA_ERR_UNSUPPORTED;
    bp->n_tokens = (size_t)p->B * p->T * p->H;
    bp->n_elems = bp->n_tokens * p->d_k;
    bp->esz = p->io_dtype == GKA_BF16 ? 2 : 4;
    // Strided q, k, v, dy are copied into the packed layout first (four tensors at the head of the workspace): every
    // kernel of the pass works on packed tensors.
    bp->strided = p->stride_b != 0 || p->stride_t != 0 || p->stride_h != 0;
    size_t off = 0;
    if (bp->strided) {
        const int64_t align = 16 / (int64_t)bp->esz;         // rows are copied 16 bytes at a time
        if (p->stride_b <= 0 || p->stride_t <= 0 || p->stride_h <= 0) return GKA_ERR_SHAPE;
        if (p->stride_h < p->d_k && p->H > 1) return GKA_ERR_SHAPE;
        if (p->stride_b % align || p->stride_t % align || p->stride_h % align) return GKA_ERR_SHAPE;
        for (int i = 0; i < 4; ++i) { bp->off_pack[i] = off; off = align_up(off + bp->n_elems * bp->esz, 256); }
    }
    for (int i = 0; i < 3; ++i) { bp->off_f32[i] = off; off = align_up(off + bp->n_elems * 4, 256); }
    for (int i = 0; i < IO_TENSORS; ++i) {
        // (float32 tensors: everything but the remainders; bf16 tensors: what the solves and the readouts hand on)
        const bool used = p->io_dtype == GKA_BF16 ? i >= IO_BF16_FIRST : i < IO_REMAINDERS;
        bp->off_io[i] = off;
        if (used) off = align_up(off + bp->n_elems * bp->esz, 256);
    }
    for (int i = 0; i < 9; ++i) { bp->off_m[i] = off; off = align_up(off + bp->n_tokens * 4, 256); }
    for (int i = 0; i < 3; ++i) {
        bp->off_fin[i] = off;
        off = align_up(off + (size_t)p->B * p->H * p->d_k * p->d_k * 4, 256);
    }
    bp->off_fwd = off;
    gka_params pf = *p;
    pf.xhat_out = nullptr;
    pf.stride_b = pf.stride_t = pf.stride_h = 0;
    Plan full, plain;                              // the plain readouts cut the scan into more segments
    if (make_plan(&pf, &full) != GKA_OK || make_plan(&pf, &plain, true) != GKA_OK) return GKA_ERR_SHAPE;
    bp->fwd_bytes = full.total > plain.total ? full.total : plain.total;
    int rs_n, rs_len;
    plan_readout_segments(p->B * p->H, (p->T + gka::kChunk - 1) / gka::kChunk, &rs_n, &rs_len);
    const size_t rbytes = align_up(gka::gla_readout_workspace_bytes(p->B * p->H, rs_n, p->d_k, p->d_v), 256);
    if (rbytes > bp->fwd_bytes) bp->fwd_bytes = rbytes;
    plan_reverse_segments(p->B * p->H, (p->T + gka::kChunk - 1) / gka::kChunk, &rs_n, &rs_len);
    const size_t vbytes = align_up(gka::reverse_workspace_bytes(p->B * p->H, rs_n, p->d_k), 256);
    if (vbytes > bp->fwd_bytes) bp->fwd_bytes = vbytes;
    const WalkRoom room = walk_room(p->B * p->H, (p->T + gka::kChunk - 1) / gka::kChunk, p->walk_chunks);
    const size_t sbytes = align_up(gka::dual_solve_workspace_bytes(room.sums, room.segs), 256);
    if (p->d_k == 128 && p->io_dtype == GKA_BF16 && sbytes > bp->fwd_bytes) bp->fwd_bytes = sbytes;
    bp->total = off + bp->fwd_bytes;
    return GKA_OK;
}
}  // namespace

size_t gka_backward_workspace_bytes(const gka_params *p)
{
    BackwardPlan bp;
    if (make_backward_plan(p, &bp) != GKA_OK) return 0;
    return bp.total;
}

gka_status gka_backward(const gka_params *p, const void *q, const void *k, const void *v, const float *gate,
                        const float *lambda, const void *dy, float *dq, float *dk, float *dv, float *dgate,
                        float *dlambda, float *dbeta, float *dalpha, void *workspace, size_t workspace_bytes,
                        void *hip_stream)
{
    return gka_backward_from_state(p, q, k, v, gate, lambda, dy, nullptr, nullptr, dq, dk, dv, dgate, dlambda, dbeta,
                                   dalpha, nullptr, nullptr, workspace, workspace_bytes, hip_stream);
}

gka_status gka_backward_from_state(const gka_params *p, const void *q, const void *k, const void *v,
                                   const float *gate, const float *lambda, const void *dy, const float *H_init,
                                   const float *U_init, float *dq, float *dk, float *dv, float *dgate,
                                   float *dlambda, float *dbeta, float *dalpha, float *dH_init, float *dU_init,
                                   void *workspace, size_t workspace_bytes, void *hip_stream)
{
    BackwardPlan bp;
    gka_status st = make_backward_plan(p, &bp);
    if (st != GKA_OK) return st;
    if (!q || !k || !v || !gate || !dy || !dq || !dk || !dv || !dgate) return GKA_ERR_NULL;
    if ((H_init == nullptr) != (U_init == nullptr)) return GKA_ERR_NULL;
    const bool with_state = H_init != nullptr || dH_init != nullptr || dU_init != nullptr;
    // initial states: bf16 tensors (the readouts that keep their state in registers), complete H_init
    if (with_state && (p->io_dtype != GKA_BF16 || p->state_layout != GKA_STATE_FULL)) return GKA_ERR_UNSUPPORTED;
    const bool rule = lambda == nullptr;          // lambda_t = lambda_scale ||H_t||_F
    if (rule && !(p->lambda_scale > 0.0f)) return GKA_ERR_NULL;
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < bp.total) return GKA_ERR_WORKSPACE;
    hipStream_t stream = (hipStream_t)hip_stream;
    unsigned char *ws = (unsigned char *)workspace;
    gka_params packed_params;
    if (bp.strided) {
        const void *src[4] = {q, k, v, dy};
        for (int i = 0; i < 4; ++i) {
            if (gka::launch_pack_rows(src[i], ws + bp.off_pack[i], p->B, p->T, p->H, p->d_k, (int)bp.esz, p->stride_b,
                                      p->stride_t, p->stride_h, stream) != hipSuccess)
                return GKA_ERR_LAUNCH;
        }
        q = ws + bp.off_pack[0]; k = ws + bp.off_pack[1]; v = ws + bp.off_pack[2]; dy = ws + bp.off_pack[3];
        packed_params = *p;
        packed_params.stride_b = packed_params.stride_t = packed_params.stride_h = 0;
        p = &packed_params;
    }
    auto io = [&](int i) { return (void *)(ws + bp.off_io[i]); };
    // (bf16 tensors without an alpha-connection: dq_t = p_t, and the solve writes it there)
    float *xf = (float *)(ws + bp.off_f32[0]);
    float *pf32 = p->io_dtype == GKA_BF16 && !p->alpha ? dq : (float *)(ws + bp.off_f32[1]);
    auto f32buf = [&](int i) { return (float *)(ws + bp.off_f32[i]); };
    float *gate_rev = (float *)(ws + bp.off_m[0]), *zeros = (float *)(ws + bp.off_m[1]), *sbuf = (float *)(ws + bp.off_m[2]);
    float *phx = (float *)(ws + bp.off_m[6]);
    float *fro = (float *)(ws + bp.off_m[3]), *cbuf = (float *)(ws + bp.off_m[4]), *Cbuf = (float *)(ws + bp.off_m[5]);
    void *fws = ws + bp.off_fwd;
    const bool io_bf16 = p->io_dtype == GKA_BF16;

    gka::BackwardGlueArgs g = {};
    g.n_elems = (int64_t)bp.n_elems; g.n_tokens = (int64_t)bp.n_tokens;
    g.T = p->T; g.H = p->H; g.d = p->d_k;
    g.q = q; g.k = k; g.v = v; g.dy = dy; g.gate = gate; g.alpha = p->alpha; g.beta = p->beta;
    g.x_f32 = xf; g.p_f32 = pf32;
    g.x_io = io(IO_X); g.xt_io = io(IO_XT); g.rhs_io = io(IO_RHS);
    g.dxt_io = io(IO_DXT); g.y_io = io(IO_Y); g.hx_io = io(IO_HX);
    g.k_rev = io(IO_KR); g.v_rev = io(IO_VR); g.dy_rev = io(IO_DYR); g.x_rev = io(IO_XR); g.p_rev = io(IO_PR);
    g.xt_rev = io(IO_XTR);
    g.gate_rev = gate_rev; g.zeros = zeros;
    g.r1 = io(IO_R1); g.r2 = io(IO_R2); g.r3 = io(IO_R3); g.r4 = io(IO_R4);
    g.dq = dq; g.dk = dk; g.dv = dv; g.dgate = dgate; g.dlambda = dlambda; g.dbeta = dbeta; g.dalpha = dalpha; g.s = sbuf;
    g.rule_a = rule ? p->lambda_scale : 0.0f; g.fro = fro; g.c = cbuf; g.C = Cbuf;
    g.vp_rev = io(IO_VPR); g.hk_io = io(IO_HK); g.r5 = io(IO_R5);

    // a forward pass with the roles given; alpha = zeros makes it the plain readout y_t = U_t q_t of the gated
    // recurrence U_t = gate_t U_{t-1} + beta_t v_t k_t^T (the solve is reduced to its starting point and discarded)
    auto fwd = [&](const void *qq, const void *kk, const void *vv, const float *gg, const float *beta,
                   const float *alpha, int n_iter, void *out, float *xhat, float *fro_out = nullptr) {
        gka_params pp = *p;                      // lambda (or its rule) as given: only the two solves use it
        pp.beta = beta; pp.alpha = alpha; pp.n_iter = n_iter; pp.xhat_out = xhat;
        pp.state_layout = GKA_STATE_FULL;
        return forward_impl(&pp, qq, kk, vv, gg, lambda, out, nullptr, nullptr, nullptr, nullptr, fro_out, fws,
                            bp.fwd_bytes, hip_stream, nullptr, alpha == zeros);
    };
    // bf16 tensors: both solves in one pass over the chunks (the second right-hand side does not depend on the first
    // solve), without U states and readout
    auto solve_both = [&](const void *q2, const void *q2_lo, float *fro_out) {
        gka_params pp = *p;
        pp.alpha = nullptr; pp.xhat_out = xf;
        pp.state_layout = GKA_STATE_FULL;
        const SecondRhs second = {q2, q2_lo, pf32, io(IO_X), io(IO_X_LO), io(IO_PR)};
        return forward_impl(&pp, q, k, v, gate, lambda, io(IO_SCRATCH), H_init, U_init, nullptr, nullptr, fro_out, fws,
                            bp.fwd_bytes, hip_stream, nullptr, false, true, &second);
    };
    auto glue = [&](int which) {
        return gka::launch_backward_glue(g, which, io_bf16, stream) == hipSuccess ? GKA_OK : GKA_ERR_LAUNCH;
    };
    // d = 128 with bf16 operands: the fused kernels' walk solves for both right-hand sides (a caller that asks for the two-phase
    // kernels or bounds their chunk states gets those). Not for sequences of one chunk in more than one round of workgroups, which
    // would each have half of their work: whole backward pass, us, walk / two-phase, 257 pairs x 64 tokens 139 / 134, x 40
    // 133 / 126, 1000 pairs x 64 311 / 304, x 40 278 / 255, x 1 226 / 213 (x 16 230 / 230); 256 pairs x 64 88 / 102, x 1 72 / 76;
    // two chunks, 257 pairs x 65 180 / 203.
    const bool walk = io_bf16 && p->d_k == 128 && p->compute == GKA_COMPUTE_BF16 && p->path == GKA_PATH_AUTO && p->slab_state_bytes == 0 &&
                      (p->T > gka::kChunk || (int64_t)p->B * p->H <= kComputeUnits);
    gka::DualSolveArgs d = {};
    if (walk) {
        gka::FusedArgs &f = d.f;
        f.q = q; f.k = k; f.v = v; f.gate = gate; f.lambda = lambda; f.fro_out = rule ? fro : nullptr;
        f.beta = p->beta; f.alpha = p->alpha; f.lambda_scale = p->lambda_scale;
        f.H_init = H_init; f.U_init = U_init;
        f.stride_h = p->d_k; f.stride_t = (int64_t)p->H * p->d_k; f.stride_b = (int64_t)p->T * p->H * p->d_k;
        f.H = p->H; f.T = p->T; f.n_iter = p->n_iter;
        f.n_pairs = p->B * p->H; f.n_chunks = (p->T + gka::kChunk - 1) / gka::kChunk;
        const WalkSegments s = plan_walk_segments(f.n_pairs, f.n_chunks, p->n_iter, p->walk_chunks);
        f.seg_len = s.seg_len; f.n_segs = s.n_segs; f.n_sums = s.n_sums; f.sums_per_seg = s.seg_len / s.sum_len;
        if (gka::dual_solve_workspace_bytes((int64_t)f.n_pairs * s.n_sums, (int64_t)f.n_pairs * s.n_segs) > bp.fwd_bytes)
            return GKA_ERR_WORKSPACE;
        d.dxt = f32buf(2);
        d.x_f32 = rule ? xf : nullptr;
        d.x_hi = io(IO_X); d.x_lo = io(IO_X_LO); d.xt_hi = io(IO_XT); d.xt_lo = io(IO_XT_LO);
        d.p_f32 = pf32; d.p_hi = io(IO_PR);
        d.dyy = sbuf;
        if (!rule) {                          // (with the rule the combination of the vectors follows)
            d.dq = p->alpha ? dq : nullptr;
            d.dlambda = dlambda; d.dalpha = dalpha;
        }
    }
    // the plain readout y_t = U_t qq_t, U_t = gate_t U_{t-1} + beta_t vv_t kk_t^T, in one kernel with the state in
    // registers (bf16 tensors); `reverse`: the recurrence runs from the last token to the first
    // (bf16 tensors: whatever operands the two solves use, the readouts take the stored bf16 tensors as they are)
    const bool fused = io_bf16;
    // out_f32: the output in float32 (the pieces of the gate gradient's sum), else in the tensors' dtype
    // q_lo, k_lo: the bf16 remainder of an operand that was computed in float32 (x), or nullptr
    // init / init_transposed: the state before the first token (forward readouts); fin: where the state after the last
    // token of the walk goes (reverse readouts: the accumulated gradient at the initial state)
    auto readout = [&](const void *qq, const void *kk, const void *vv, const float *beta, bool reverse, void *out,
                       int seg_mode = 0, float *out_f32 = nullptr, const void *q_lo = nullptr,
                       const void *k_lo = nullptr, const float *init = nullptr,
                       bool init_transposed = false, float *fin = nullptr, const float *dot_with = nullptr,
                       float *dot_out = nullptr) {
        gka::ReadoutArgs r = {};                     // (optional pointers default to nullptr)
        r.init_state = init; r.init_transposed = init_transposed; r.final_state = fin;
        r.dot_with = dot_with; r.dot_out = dot_out;
        r.q = qq; r.q_lo = q_lo; r.k_lo = k_lo; r.q_is_f32 = false; r.k = kk; r.v = vv; r.o = out;
        r.o_f32 = out_f32;
        r.gate = gate; r.beta = beta;
        r.stride_h = p->d_k; r.stride_t = (int64_t)p->H * p->d_k; r.stride_b = (int64_t)p->T * p->H * p->d_k;
        r.qk_stride_h = r.stride_h; r.qk_stride_t = r.stride_t; r.qk_stride_b = r.stride_b;
        r.H = p->H; r.T = p->T; r.n_pairs = p->B * p->H;
        plan_readout_segments(r.n_pairs, (p->T + gka::kChunk - 1) / gka::kChunk, &r.n_segs, &r.seg_len);
        if (seg_mode >= 2) {                         // the summaries of the solves' walk
            r.n_segs = d.f.n_sums;
            r.seg_len = d.f.seg_len / d.f.sums_per_seg;
        }
        r.seg_buf = (float *)fws;
        r.seg_logdecay = r.seg_buf + (size_t)r.n_pairs * r.n_segs * (seg_mode >= 2 ? gka::kSummaryPlanes : 1) * p->d_k * p->d_v;
        r.reverse = reverse; r.seg_mode = seg_mode;
        return gka::launch_gla_readout(r, p->d_k, p->d_v, stream) == hipSuccess ? GKA_OK : GKA_ERR_LAUNCH;
    };
    g.natural_order = fused;
    if (walk && !rule) g.dyy = sbuf;          // (the combination reads and replaces it token by token)
    if (fused) {
        g.dxt_io = f32buf(2);                     // (float32)
        g.phx = phx; g.kd = (float *)(ws + bp.off_m[7]); g.vd = (float *)(ws + bp.off_m[8]);
        // bf16 tensors: the second solve takes alpha dxt, and the readouts take x and xt, as value + remainder
        g.rhs_lo_io = io(IO_RHS_LO); g.xt_lo_io = io(IO_XT_LO);
    }
#define GKA_TRY(expr) do { gka_status e_ = (expr); if (e_ != GKA_OK) return e_; } while (0)
    if (fused) {
        // dxt_t = U_t^T dy_t: the recurrence with the roles of k and v exchanged, read out with dy. (alpha_t dxt_t in bf16 from
        // the readout itself: 97 -> 152 us at 64 pairs x 4096 tokens, its own pass over memory takes 41.)
        // (With the solves' walk the readouts start from its summaries: of U^T here, of H below; a summary launch less for each.)
        if (walk && gka::launch_dual_solve_summaries(d, fws, stream) != hipSuccess) return GKA_ERR_LAUNCH;
        GKA_TRY(readout(dy, v, k, p->beta, false, nullptr, walk ? 2 : 0, f32buf(2), nullptr, nullptr, U_init, true));
        // x_t = CH(H_t + lambda_t I, q_t, r) and p_t = CH(H_t + lambda_t I, alpha_t dxt_t, r)
        if (walk) {
            if (gka::launch_dual_solve(d, fws, stream) != hipSuccess) return GKA_ERR_LAUNCH;
        } else {
            GKA_TRY(glue(1));
            GKA_TRY(solve_both(io(IO_RHS), io(IO_RHS_LO), rule ? fro : nullptr));
            // xt in the tensors' dtype (x and p have been written so by the solve)
            if (p->alpha) GKA_TRY(glue(0));
        }
        // p_t . H_t x_t
        GKA_TRY(readout(io(IO_X), k, k, p->beta, false, nullptr, walk ? 3 : 0, nullptr, io(IO_X_LO), nullptr, H_init, false,
                        nullptr, pf32, phx));
    } else {
        // the forward solve and output; then x, xt in the tensors' dtype, the all-zero alpha and the reversed gates
        GKA_TRY(fwd(q, k, v, gate, p->beta, p->alpha, p->n_iter, io(IO_Y), xf, rule ? fro : nullptr));
        GKA_TRY(glue(0));
        GKA_TRY(fwd(dy, v, k, gate, p->beta, zeros, 0, io(IO_DXT), nullptr));
        GKA_TRY(glue(1));
        GKA_TRY(fwd(io(IO_RHS), k, v, gate, p->beta, nullptr, p->n_iter, io(IO_SCRATCH), pf32));
        GKA_TRY(fwd(io(IO_X), k, k, gate, p->beta, zeros, 0, io(IO_HX), nullptr));
    }
    // the rule's extra gradient -c_t H_t at every state: c_t, C_t = sum_{s>=t} M[t,s]^2 c_s, and H_t k_t
    if (rule) {
        GKA_TRY(glue(5));
        GKA_TRY(glue(6));
        if (fused) GKA_TRY(readout(k, k, k, p->beta, false, io(IO_HK), walk ? 3 : 1, nullptr, nullptr, nullptr, H_init));
        else GKA_TRY(fwd(k, k, k, gate, p->beta, zeros, 0, io(IO_HK), nullptr));
    }
    // reverse recurrences: A_t k_t, A_t^T k_t, Ubar_t^T v_t, Ubar_t k_t (no write gate inside them)
    if (!fused || rule) GKA_TRY(glue(2));
    if (fused) {
        float *fin_px = with_state ? (float *)(ws + bp.off_fin[0]) : nullptr;
        float *fin_xtdy = with_state ? (float *)(ws + bp.off_fin[1]) : nullptr;
        float *fin_ck = with_state && rule ? (float *)(ws + bp.off_fin[2]) : nullptr;
        if (rule) GKA_TRY(readout(k, k, io(IO_VPR), nullptr, true, io(IO_R5), 0, nullptr, nullptr, nullptr, nullptr, false,
                                  fin_ck));
        g.fin_px = fin_px; g.fin_xtdy = fin_xtdy; g.fin_ck = fin_ck;
        // (the gradient at the initial H needs A_t = sum M[t,s] p_s x_s^T itself at token 0, not its symmetric part; the
        // readout's output is not wanted)
        if (dH_init) GKA_TRY(readout(k, io(IO_X), io(IO_PR), nullptr, true, io(IO_SCRATCH), 0, nullptr, nullptr, io(IO_X_LO),
                                     nullptr, false, fin_px));
        gka::ReverseArgs rv = {};
        rv.k = k; rv.v = v; rv.dy = dy; rv.p = io(IO_PR); rv.x = io(IO_X); rv.x_lo = io(IO_X_LO);
        rv.gate = gate; rv.beta = p->beta;
        rv.dk = dk; rv.dv = dv; rv.kd = (float *)(ws + bp.off_m[7]); rv.vd = (float *)(ws + bp.off_m[8]);
        rv.fin_xtdy = fin_xtdy;
        rv.H = p->H; rv.T = p->T; rv.n_pairs = p->B * p->H;
        plan_reverse_segments(rv.n_pairs, (p->T + gka::kChunk - 1) / gka::kChunk, &rv.n_segs, &rv.seg_len);
        rv.seg_buf = (float *)fws;
        rv.seg_logdecay = rv.seg_buf + (size_t)rv.n_pairs * rv.n_segs * 2 * p->d_k * p->d_k;
        if (!p->alpha) {                          // xt = x
            if (gka::launch_reverse(rv, p->d_k, 3, stream) != hipSuccess) return GKA_ERR_LAUNCH;
        } else {
            if (gka::launch_reverse(rv, p->d_k, 1, stream) != hipSuccess) return GKA_ERR_LAUNCH;
            rv.x = io(IO_XT); rv.x_lo = io(IO_XT_LO);
            if (gka::launch_reverse(rv, p->d_k, 2, stream) != hipSuccess) return GKA_ERR_LAUNCH;
        }
    } else {
        if (rule) GKA_TRY(fwd(io(IO_KR), io(IO_KR), io(IO_VPR), gate_rev, nullptr, zeros, 0, io(IO_R5), nullptr));
        GKA_TRY(fwd(io(IO_KR), io(IO_XR), io(IO_PR), gate_rev, nullptr, zeros, 0, io(IO_R1), nullptr));
        GKA_TRY(fwd(io(IO_KR), io(IO_PR), io(IO_XR), gate_rev, nullptr, zeros, 0, io(IO_R2), nullptr));
        GKA_TRY(fwd(io(IO_VR), io(IO_DYR), io(IO_XTR), gate_rev, nullptr, zeros, 0, io(IO_R3), nullptr));
        GKA_TRY(fwd(io(IO_KR), io(IO_XTR), io(IO_DYR), gate_rev, nullptr, zeros, 0, io(IO_R4), nullptr));
    }
    GKA_TRY(glue(3));
    GKA_TRY(glue(4));
    if (dH_init || dU_init) {
        g.H_init = H_init; g.dH_init = dH_init; g.dU_init = dU_init; g.n_pairs = p->B * p->H;
        GKA_TRY(glue(7));
    }
#undef GKA_TRY
    return GKA_OK;
}

// ---- latent sketching: down-projection, the solve in the sketched space (up to 32 dimensions on the kernels of
// gka_small_dim.hip, else in 64 zero-padded dimensions on the forward kernels), readout in the sketched space (d = 128)
// or up-projection and plain readout with the full U_t (d = 64)
namespace {
struct SketchPlan {
    size_t n_tokens;
    size_t off_qs, off_ks, off_scratch, off_z, off_xhat, off_xhat_lo, off_fwd, fwd_bytes, total;
    gka_params inner;             // the solve's problem: d = 64, packed
    int rs_n, rs_len;
    bool small;                   // d_s <= 32: the solve runs on the kernels of gka_small_dim.hip
};
constexpr int kSketchDim = 64;
constexpr int kSketchSmall = 32;
gka_status make_sketch_plan(const gka_params *p, int d_s, SketchPlan *sp)
{
    gka_status s = check_common(p, false);
    if (s != GKA_OK) return s;
    if (p->io_dtype != GKA_BF16 || p->compute != GKA_COMPUTE_BF16) return GKA_ERR_UNSUPPORTED;
    if (!chunked_dim(p->d_k) || p->path == GKA_PATH_RECURRENT) return GKA_ERR_UNSUPPORTED;
    if (p->stride_b != 0 || p->stride_t != 0 || p->stride_h != 0) return GKA_ERR_UNSUPPORTED;
    if (p->phase != GKA_PHASE_ALL || p->alpha) return GKA_ERR_UNSUPPORTED;
    if (d_s < 1 || d_s > kSketchDim) return GKA_ERR_SHAPE;
    sp->n_tokens = (size_t)p->B * p->T * p->H;
    sp->inner = *p;
    sp->inner.d_k = sp->inner.d_v = kSketchDim;
    sp->inner.xhat_out = nullptr;
    sp->inner.state_layout = GKA_STATE_FULL;
    size_t off = 0;
    sp->off_qs = off; off = align_up(off + sp->n_tokens * kSketchDim * 2, 256);
    sp->off_ks = off; off = align_up(off + sp->n_tokens * kSketchDim * 2, 256);
    sp->off_scratch = off; off = align_up(off + sp->n_tokens * kSketchDim * 2, 256);
    sp->off_z = off; off = align_up(off + sp->n_tokens * kSketchDim * 4, 256);
    sp->off_xhat = off; off = align_up(off + sp->n_tokens * p->d_k * 2, 256);
    sp->off_xhat_lo = off; off = align_up(off + sp->n_tokens * p->d_k * 2, 256);
    sp->off_fwd = off;
    Plan pl;
    if (make_plan(&sp->inner, &pl) != GKA_OK) return GKA_ERR_SHAPE;
    sp->fwd_bytes = pl.total;
    plan_readout_segments(p->B * p->H, (p->T + gka::kChunk - 1) / gka::kChunk, &sp->rs_n, &sp->rs_len);
    const size_t rbytes = align_up(gka::gla_readout_workspace_bytes(p->B * p->H, sp->rs_n, p->d_k, p->d_v), 256);
    if (rbytes > sp->fwd_bytes) sp->fwd_bytes = rbytes;
    // up to 32 sketched dimensions the solve has kernels of its own (their chunk states: 2 x 4 KiB per chunk)
    sp->small = d_s <= kSketchSmall;
    if (sp->small) {
        const size_t sbytes = gka::small_dim_workspace_bytes(p->B * p->H, (p->T + gka::kChunk - 1) / gka::kChunk, kSketchSmall, false);
        if (sbytes > sp->fwd_bytes) sp->fwd_bytes = sbytes;
    }
    sp->total = off + sp->fwd_bytes;
    return GKA_OK;
}
}  // namespace

size_t gka_forward_sketched_workspace_bytes(const gka_params *p, int d_s)
{
    SketchPlan sp;
    if (make_sketch_plan(p, d_s, &sp) != GKA_OK) return 0;
    return sp.total;
}

gka_status gka_forward_sketched(const gka_params *p, const void *q, const void *k, const void *v, const float *gate,
                                const float *lambda, const float *S, int d_s, int sketch_per_head, void *o,
                                void *workspace, size_t workspace_bytes, void *hip_stream)
{
    SketchPlan sp;
    gka_status st = make_sketch_plan(p, d_s, &sp);
    if (st != GKA_OK) return st;
    if (!q || !k || !v || !gate || !S || !o) return GKA_ERR_NULL;
    if (!lambda && !(p->lambda_scale > 0.0f)) return GKA_ERR_NULL;
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < sp.total) return GKA_ERR_WORKSPACE;
    hipStream_t stream = (hipStream_t)hip_stream;
    unsigned char *ws = (unsigned char *)workspace;
    gka::SketchArgs sa = {};
    // stored width of the sketched tensors: 32 where everything downstream works in 32 dimensions
    const int sw = sp.small && p->d_v == 128 ? kSketchSmall : kSketchDim;
    sa.q = q; sa.k = k; sa.S = S; sa.d_s = d_s; sa.per_head = sketch_per_head != 0; sa.out_width = sw;
    sa.qs = ws + sp.off_qs; sa.ks = ws + sp.off_ks; sa.z = (const float *)(ws + sp.off_z);
    sa.xhat_hi = ws + sp.off_xhat; sa.xhat_lo = ws + sp.off_xhat_lo;
    sa.T = p->T; sa.H = p->H;
    const int n_pairs = p->B * p->H;
    if (gka::launch_sketch(sa, n_pairs, p->d_k, false, stream) != hipSuccess) return GKA_ERR_LAUNCH;
    // z_t = CH(S H_t S^T + lambda_t I, S q_t, r): the forward pass on the sketched keys and queries, its own readout
    // discarded (the sketched keys stand in for its values)
    if (sp.small) {
        gka::SmallArgs ss = {};                  // (no values, no output: the solve alone)
        ss.q = sa.qs; ss.k = sa.ks;
        ss.stride_h = sw; ss.stride_t = (int64_t)p->H * sw; ss.stride_b = (int64_t)p->T * p->H * sw;
        ss.d = kSketchSmall;
        ss.gate = gate; ss.lambda = lambda; ss.beta = p->beta; ss.lambda_scale = p->lambda_scale;
        ss.xhat_out = (float *)(ws + sp.off_z); ss.xhat_row = sw;
        ss.xhat_zero_upper = sw == kSketchDim;   // (the up-projection of the d = 64 path reads all 64 stored features)
        ss.T = p->T; ss.H = p->H; ss.n_pairs = n_pairs; ss.n_chunks = (p->T + gka::kChunk - 1) / gka::kChunk;
        ss.n_iter = p->n_iter;
        if (gka::launch_small_dim_forward(ss, ws + sp.off_fwd, stream) != hipSuccess) return GKA_ERR_LAUNCH;
    } else {
        gka_params inner = sp.inner;
        inner.xhat_out = (float *)(ws + sp.off_z);
        st = forward_impl(&inner, sa.qs, sa.ks, sa.ks, gate, lambda, ws + sp.off_scratch, nullptr, nullptr, nullptr,
                          nullptr, nullptr, ws + sp.off_fwd, sp.fwd_bytes, hip_stream, nullptr, false, true);
        if (st != GKA_OK) return st;
    }
    gka::ReadoutArgs r = {};                     // (optional pointers default to nullptr)
    r.k_lo = nullptr;
    r.v = v; r.o = o; r.o_f32 = nullptr; r.gate = gate; r.beta = p->beta;
    r.stride_h = p->d_v; r.stride_t = (int64_t)p->H * p->d_v; r.stride_b = (int64_t)p->T * p->H * p->d_v;
    r.H = p->H; r.T = p->T; r.n_pairs = n_pairs;
    r.n_segs = sp.rs_n; r.seg_len = sp.rs_len;
    r.seg_buf = (float *)(ws + sp.off_fwd);
    r.reverse = false; r.seg_mode = 0;
    if (p->d_v == 128) {
        // y_t = U_t S^T z_t = (sum_i eta_{t,i} beta_i v_i (S k_i)^T) z_t: the readout runs in the sketched space, on the
        // stored sketched keys and the float32 z_t (split into value + remainder inside the kernel), with a d_v x 64
        // state; the projected solution xhat_t is never formed
        r.q = sa.z; r.q_lo = nullptr; r.q_is_f32 = true; r.k = sa.ks;
        r.qk_stride_h = sw; r.qk_stride_t = (int64_t)p->H * sw;
        r.qk_stride_b = (int64_t)p->T * p->H * sw;
        r.seg_logdecay = r.seg_buf + (size_t)n_pairs * r.n_segs * kSketchDim * p->d_v;
        // (up to 32 sketched dimensions: a d_v x 32 state on the first 32 stored features)
        return gka::launch_gla_readout(r, sp.small ? kSketchSmall : kSketchDim, p->d_v, stream) == hipSuccess
                   ? GKA_OK : GKA_ERR_LAUNCH;
    }
    // d = 64: xhat_t = S^T z_t as value + remainder, then y_t = U_t xhat_t with the state of Eq. (CH)
    if (gka::launch_sketch(sa, n_pairs, p->d_k, true, stream) != hipSuccess) return GKA_ERR_LAUNCH;
    r.q = sa.xhat_hi; r.q_lo = sa.xhat_lo; r.q_is_f32 = false; r.k = k;
    r.qk_stride_h = r.stride_h; r.qk_stride_t = r.stride_t; r.qk_stride_b = r.stride_b;
    r.seg_logdecay = r.seg_buf + (size_t)n_pairs * r.n_segs * p->d_k * p->d_v;
    return gka::launch_gla_readout(r, p->d_k, p->d_v, stream) == hipSuccess ? GKA_OK : GKA_ERR_LAUNCH;
}

const char *gka_status_string(gka_status s)
{
    switch (s) {
    case GKA_OK: return "ok";
    case GKA_ERR_NULL: return "required pointer is NULL";
    case GKA_ERR_SHAPE: return "invalid size or stride";
    case GKA_ERR_UNSUPPORTED: return "unsupported head dimension, chunk, dtype or compute mode";
    case GKA_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case GKA_ERR_LAUNCH: return "HIP launch failed";
    case GKA_ERR_STATIC_SCRATCH: return "problem needs more scratch than gka_forward_static's fixed array holds";
    }
    return "unknown status";
}

int gka_version(void) { return 810; }

}  // extern "C"
