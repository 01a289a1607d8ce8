// Internal launch interface between the C-ABI host layer and the gfx950 kernels.
// Every launcher enqueues on `st` and returns the hipError_t of the launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace icarus {

typedef uint16_t bf16_raw;  // raw bfloat16 bits

struct Dims {
    int d, Hq, Hkv, D, F, Bk, M, r;
    int bf16;      // storage type: 1 = bfloat16, 0 = float32
    int kv8;       // 1: the KV pool holds FP8 E4M3 codes, value = code * k_scale (K plane) or v_scale (V plane)
    float k_scale, v_scale;
    int qk_norm;
    double theta;
    float eps, lora_scale;
};

// Per-call row metadata, device int32 arrays.
struct RowMeta {
    const int32_t *row_seq;    // [R] sequence of each row
    const int32_t *row_model;  // [R] -1 = logical encoder row, else adapter id
    const int32_t *row_pos;    // [R] position of the row's token
    const int32_t *row_kvlen;  // [R] cache positions the row attends to (0..kvlen-1)
    const int32_t *order = nullptr;  // decode with adapters: rows for the workgroups of the row kernels, see row_order
    int n_order = 0;
    const int32_t *rope_tiles = nullptr;  // prefill: the rows in tiles for launch_rope_append_tiles
    int n_rope_tiles = 0;
};

// ---- generic vector kernels (any shape; fp32 accumulation) -------------------------------
// y[r,:] = x[r,:] * rsqrt(mean(x^2)+eps) * w        (storage type in and out)
hipError_t launch_rmsnorm(const Dims &dm, const void *x, const void *w, void *y, int R, int n, hipStream_t st);
// Y[m, n] (fp32, ld = ldy) = sum_k X[m,k] W[n,k];  X, W storage type
hipError_t launch_gemm_generic(const Dims &dm, const void *X, int ldx, const void *W, int M, int N, int K,
                               float *Y, int ldy, hipStream_t st);
// t[row, 0..r) (fp32) = lora_scale * A[model(row)] x[row]   for decoder rows (model >= 0)
hipError_t launch_lora_shrink_generic(const Dims &dm, const void *X, int ldx, const void *A, int K,
                                      const int32_t *row_model, float *t, int R, hipStream_t st);
// Y[row, n] += sum_k B[model(row)][n,k] t[row,k]           for decoder rows
hipError_t launch_lora_expand_generic(const Dims &dm, const float *t, const void *B, int N,
                                      const int32_t *row_model, float *Y, int ldy, int R, hipStream_t st);
// out[r, n] (storage) = resid[r, n] (storage) + acc[r, n] (fp32)
hipError_t launch_resid_store(const Dims &dm, const void *resid, const float *acc, void *out, int R, int n, hipStream_t st);
// h[r, n] (storage) = silu(gate[r,n]) * up[r,n]     (fp32 in)
hipError_t launch_silu_mul(const Dims &dm, const float *gate, const float *up, void *h, int R, int n, hipStream_t st);
// QK-RMSNorm (optional) + RoPE on q (all rows) and k (encoder rows), q -> q_out (storage, [R,Hq,D]),
// k, v of encoder rows -> paged cache; slot_out[slot_by_row ? row : seq] = slot.
// qkv: fp32 [R, ldq] with q at column 0, k at Hq*D, v at (Hq+Hkv)*D, given as `splits` slices that are
// summed (`slice` floats apart; splits = 1: the plain array).
hipError_t launch_rope_append(const Dims &dm, const float *qkv, int ldq, int splits, size_t slice, const RowMeta &rm,
                              const int32_t *bt, int max_blocks, void *pool, void *q_out, int64_t *slot_out, int slot_by_row,
                              const void *q_norm, const void *k_norm, int R, hipStream_t st, const int32_t *row_map = nullptr);
// The same for encoder rows only, head_dim 128 and blocks of 16, by tiles of consecutive rows within one KV block: tiles (device)
// = first row | rows << 16.  kv_only: q is neither read nor written.  slot_out is by row.
bool rope_tiles_supported(const Dims &dm, int ldq, size_t slice);
bool rope_tiles_pay(const Dims &dm, int rows, int n_tiles);
hipError_t launch_rope_append_tiles(const Dims &dm, const float *qkv, int ldq, int splits, size_t slice, const RowMeta &rm,
                                    const int32_t *tiles, int n_tiles, bool kv_only, const int32_t *bt, int max_blocks, void *pool,
                                    void *q_out, int64_t *slot_out, const void *q_norm, const void *k_norm, hipStream_t st);
// Cosines and sines [R][64] of the rows' angles and their slots [R], for launch_gemm_qkv.
hipError_t launch_rope_table(const Dims &dm, const RowMeta &rm, const int32_t *bt, int max_blocks, int R, float *cs, float *sn, int64_t *slot,
                             hipStream_t st);
// out[row, h, :] = softmax(q[row,h,:] K^T / sqrt(D)) V over positions 0..row_kvlen[row]-1 of row_seq[row]
hipError_t launch_attn_generic(const Dims &dm, const void *q, const void *pool, const int32_t *bt, int max_blocks,
                               const RowMeta &rm, void *out, int R, hipStream_t st);

// ---- the same for at most kSkinnyRows rows (skinny_kernels.hip) ---------------------------------
constexpr int kSkinnyRows = 16;
enum { SKINNY_F32 = 0, SKINNY_RESID = 1, SKINNY_DUAL = 2 };  // float out; storage out + residual; silu(gate) * up, storage out
struct SkinnyGemm {
    const void *X; int ldx, R, K;             // storage type
    const void *W[3]; int n[3];               // up to three weight segments [n, K] stacked along the outputs; DUAL: gate, up (n[0] each)
    const void *B[2]; const float *t;         // adapter B [M, n[0], r] of segment 0 (DUAL: gate, up), t [targets][R][r]; null: none
    const int32_t *row_model;
    const void *resid; void *Y; int ldy;      // SKINNY_RESID: resid has the stride of Y
    int mode;
    // In place of launch_row_generic before it, where skinny_takes_rows (else both null): the rows are rmsnorm(X) * wn (not of
    // SKINNY_RESID), and t = lora_scale * A[model(row)] x of the targets that B names
    const void *wn, *A[2];
};
bool skinny_takes_rows(const Dims &dm, const SkinnyGemm &g);
hipError_t launch_gemm_skinny(const Dims &dm, const SkinnyGemm &g, hipStream_t st);
// y = rmsnorm(x) * wn (wn != null) and, with A0, t[target][row][0..r) = lora_scale * A_target[model(row)] (y or x)
hipError_t launch_row_generic(const Dims &dm, const void *x, int ldx, int K, const void *wn, void *y, const void *A0, const void *A1,
                              const int32_t *row_model, float *t, int R, hipStream_t st);

// plain grid-stride copy of `bytes` bytes (multiple of 16), kernel k_bench_copy: profiler calibration
hipError_t launch_bench_copy(const void *src, void *dst, size_t bytes, hipStream_t st);
// streaming read of `bytes` bytes (whole 8 KB chunks) by kernel k_bench_read: the read rate HBM sustains; out: one word
hipError_t launch_bench_read(const void *src, size_t bytes, uint32_t *out, hipStream_t st);
// register-resident MFMA loop, kernel k_bench_mfma: waves (multiple of 4) x iters x 8 MFMAs 32x32x16 bf16
hipError_t launch_bench_mfma(float *out, int waves, int iters, hipStream_t st);

// ---- matrix-core kernels (bf16 storage) ------------------------------------------------------
// Host-built plan of the attention kernels.  All arrays are device int32.
// Decode (causal = 0): the call's work -- the cached tokens of every sequence -- is laid on one line
// and cut into n_wgs equal shares; share b is walked by Hkv workgroups (one per kv-head), each over
// piece b and the pieces from share_next[b] on up to one that is marked last, a piece being a token range of one sequence.  Piece
// boundaries are multiples of 32 tokens.  A sequence cut into several pieces leaves one partial
// result per piece and kv-head.  Arrays: pieces, share_next, and of the sequences row0, part0, nparts.
// Prefill (causal = 1): one workgroup per piece and kv-head; a piece is the whole walk of a token group, or a part of
// it that leaves a partial result (launch_attn_merge combines them).  Inner boundaries on whole rounds of the walk.
// Without any cut walk the arrays of parts are null: item_begin, _len, _part, _direct, seq_part0, _nparts.
constexpr int kPieceDirect = 1 << 30, kPieceLast = 1 << 29, kPieceTokens = kPieceLast - 1;  // direct: the piece is its whole sequence; last: of its share
struct AttnPlan {
    const int32_t *item_seq;     // [n_items] plan sequence of the piece
    const int32_t *item_begin;   // [n_items] first token of the piece
    const int32_t *item_len;     // [n_items] tokens of the piece
    const int32_t *item_part;    // [n_items] partial-result slot of the piece
    const int32_t *item_direct;  // [n_items] 1: the piece is its whole sequence: write the final output
    const int32_t *pieces;       // decode: [n_items][5] first row | rows << 16, row of the block table, first token, tokens | kPieceDirect | kPieceLast, partial-result slot
    const int32_t *share_next;   // decode: [n_wgs] second piece of each share
    const int32_t *seq_kvlen;    // [S] tokens to attend to
    const int32_t *seq_row0;     // [S] first row of the sequence
    const int32_t *seq_rows;     // [S] rows (stacked streams) of the sequence
    const int32_t *seq_part0;    // [S] first partial slot
    const int32_t *seq_nparts;   // [S] number of pieces
    const int32_t *seq_bt;       // [S] row of the block table the sequence reads
    int n_seq;                         // S
    int n_items, n_wgs, chunk, g_max;  // n_wgs: shares; chunk: longest piece; g_max: largest stacked group (rows * Hq/Hkv)
    int causal;                  // 1: row t of a sequence attends to kv_len - (rows - 1 - t) tokens (prefill)
    int pipelined;               // prefill: see attn_prefill_pipelined
};
// ICaRusLinear GEMM on matrix cores.  Y = X W^T (+ T Bcat^T), see gemm_mfma.hip.
enum { GEMM_PLAIN = 0, GEMM_DUAL = 1 };          // DUAL: W[0] = gate, W[1] = up, Y = silu(gate) * up
enum { EPI_F32 = 0, EPI_BF16_RESID = 1 };        // plain epilogues (DUAL always stores bf16)
enum TileKind { TILE_AUTO = 0, TILE_64x128, TILE_128, TILE_192x128, TILE_256x256, TILE_192x256, TILE_160x256, TILE_KINDS };
struct GemmArgs {
    const bf16_raw *X; int ldx; int R; int K;    // activations [R, K] (row stride ldx)
    const bf16_raw *W[3]; int n_seg[3]; int nseg; // weight segments stacked along N, each [n_seg, K]
    const bf16_raw *T; int ldt;                  // masked shrink result [R, ldt] or null
    const bf16_raw *B[2]; int r; int M_models;   // adapter B [M, n_seg[0], r] of segment 0 (DUAL: gate, up)
    int mode, epi;
    void *Y; int ldy;                            // EPI_F32: float [splits][slice_rows][ldy]; else bf16 [R][ldy]
    int slice_rows;                              // R at least (0: R)
    const bf16_raw *resid; int ldr;              // EPI_BF16_RESID: added to the result
    int splits;                                  // split-K slices (EPI_F32 without adapters only)
    int tile;                                    // tile kind (TILE_AUTO: chosen by the launcher)
    // filled by the launcher
    int tiles_seg[3]; int m_tiles, n_tiles, K_ext, k_per_split;
    int panel_m, panel_n, panels_m, n_panels;       // tile order: panels of panel_m x panel_n tiles (n_panels per K slice)
    uint32_t inv_panels, inv_panels_m, inv_panel_m; // gemm_inv of n_panels, panels_m, panel_m
    // Grouped launch (optional): row_tiles, device [n_row_tiles][3] = first row, end row, group of each row tile (gemm_tile_rows
    // rows at most).  Group 0 multiplies W[0] (DUAL: W[0], W[1]), group j > 0 Wg[.] + (j - 1) * wg_stride elements.
    const int32_t *row_tiles; int n_row_tiles;
    const bf16_raw *Wg[2]; size_t wg_stride;
    uint32_t stagger;                                // gemm_inv of a slice's slabs of base weights, 0: every workgroup starts at the first one (gemm_staggered)
};
bool gemm_mfma_supported(const Dims &dm, int K);
// fills the tile order from m_tiles, n_tiles and splits, for bm x bn tiles and per_cu workgroups to a CU
void gemm_set_panels(GemmArgs *g, int bm, int bn, int per_cu);
// grid of the launch: x = place in a panel * 8 + XCD, y = panels of an XCD in turn
inline dim3 gemm_grid(const GemmArgs &g) {
    return dim3((unsigned)(g.panel_m * g.panel_n * 8), (unsigned)((g.n_panels * g.splits + 7) / 8));
}
// x / n for x * n < 2^32, by the host's inv = ceil(2^32 / n) (0 for n = 1): a division would cost these short kernels
// as much as a dozen loads.  Without a branch, so that the arguments of a whole tile_at are loaded at once: one after the
// other behind branches they made the small decode launches 0.2 us longer (10.0 -> 10.3).
inline uint32_t gemm_inv(int n) { return n > 1 ? (uint32_t)((((uint64_t)1 << 32) + (uint64_t)n - 1) / (uint64_t)n) : 0u; }
__host__ __device__ __forceinline__ int gemm_div(int x, uint32_t inv) { return (int)(((uint64_t)(uint32_t)x * inv) >> 32) + (x & -(int)(inv == 0)); }
// Tile and K slice of workgroup (bx, by); false: none.  Neighbouring columns of a panel go to one XCD.  Dealing the columns
// of a single row tile over the XCDs instead depends on how the weight rows' strides fall: a step of 32 rows with an LM head
// of 4096 -> 128256 425 -> 414 us, but with one of 4096 -> 65536 281 -> 322 us, and 9 rows of gate and up, 8192 -> 2 x 28672,
// 177 -> 227 us.
__host__ __device__ __forceinline__ bool tile_at(const GemmArgs &g, int bx, int by, int *tile_m, int *tile_n, int *kz) {
    const int within = bx >> 3, p = by * 8 + (bx & 7);
    *kz = gemm_div(p, g.inv_panels);
    const int panel = p - *kz * g.n_panels;
    const int pn = gemm_div(panel, g.inv_panels_m), wn = gemm_div(within, g.inv_panel_m);
    *tile_m = (panel - pn * g.panels_m) * g.panel_m + within - wn * g.panel_m;
    *tile_n = pn * g.panel_n + wn;
    return (*kz < g.splits) & (*tile_m < g.m_tiles) & (*tile_n < g.n_tiles);
}
__device__ __forceinline__ bool tile_of_workgroup(const GemmArgs &g, int *tile_m, int *tile_n, int *kz) {
    return tile_at(g, blockIdx.x, blockIdx.y, tile_m, tile_n, kz);
}
hipError_t launch_gemm_mfma(GemmArgs g, hipStream_t st);
// QKV projection of encoder rows (head_dim 128, blocks of 16, no adapters) that normalises and rotates in its epilogue and writes q and
// the cache itself; a whole launch in tiles of k_gemm_quad (gemm_qkv_fused).
struct QkvStore {
    const float *cs, *sn; const int64_t *slot;   // of each row, see launch_rope_table
    bf16_raw *q; void *pool;
    const bf16_raw *q_norm, *k_norm;             // null: no QK-norm
    int Hq, Hkv, kv8; float eps, k_scale, v_scale;
};
bool gemm_qkv_fused(const GemmArgs &g, struct GemmPlan plan);
hipError_t launch_gemm_qkv(GemmArgs g, const QkvStore &e, hipStream_t st);
hipError_t launch_gemm_quad_qkv(const GemmArgs &g, const QkvStore &e, hipStream_t st);
// How a GEMM is run: tile kind and split-K slices, at most max_splits (1 where K cannot be split: DUAL).  takes_slices: a
// later kernel of the caller reads the slices as they are, no reduction is launched for them.
struct GemmPlan { int tile, splits; };
GemmPlan gemm_plan(const GemmArgs &g, int max_splits, bool takes_slices);
// Grouped launches: tile kind for groups of rows [off[j], off[j + 1]), its height, and the K slices to use.
int gemm_row_tile(const int *off, int n_groups);
int gemm_tile_rows(int tile);
int gemm_tile_cols(int tile);
int gemm_grouped_splits(const GemmArgs &g, int max_splits, bool takes_slices);
bool gemm_tile_marked(int tile);  // the mark of 192 and 160 rows by 256 in icarus_gemm_choice and icarus_gemm: part of their name, chooses nothing
// Tiles of gemm_quad.hip: 256, 192 or 160 rows by 256, and 192 (or 160 or 128, where as many hold the rows) by 128; launch_gemm_mfma takes this
// path for them.  g.K_ext and g.k_per_split are set.
constexpr int kQuadMaxK = 1 << 23;  // a row's offset within its tile is kept in 32 bits of bytes
hipError_t launch_gemm_quad(const GemmArgs &g, hipStream_t st);
// Sum split-K partials P[splits][R][N] (fp32) and apply the epilogue `epi` into Y.
hipError_t launch_splitk_reduce(const float *P, int splits, int R, int N, int epi, void *Y, int ldy, const void *resid,
                                int ldr, hipStream_t st);
// Row-wise kernels (bf16 storage).  T [R, targets*M*r] (bf16) is the masked LoRA shrink the GEMM reads
// as extra K columns: T[row, t*M*r + j*r + i] = lora_scale * (A_t[j] x_row)_i for j = row_model[row], zero
// in every other column (encoder rows: all zero).  A: [M][r][K].
bool row_shrink_supported(int r, int targets);
// Order of the rows over the workgroups of the kernels below: entry = row | (model + 1) << 16, -1: none; at most R + 16 entries,
// a multiple of 8.  Returns how many; 0: few rows, or a model that an entry does not hold: the rows in the order they have.
int row_order(const int32_t *row_model, int R, int32_t *order);
// y = rmsnorm(x) * wn for R rows of K, and (A0 != null) the shrink of y for one or two targets that
// share y; also sets zero[0..n_zero) = 0.
hipError_t launch_norm_shrink(const Dims &dm, const void *x, const void *wn, void *y, int R, int K, const void *A0, const void *A1,
                              const RowMeta &rm, void *T, int *zero, int n_zero, hipStream_t st);
// the same on rows that are still in pieces: xsum = resid + sum of `splits` fp32 slices [R, K] (`slice` floats
// apart, the split-K partials of the projection before the norm) is formed, rounded, stored, and normalised
hipError_t launch_sum_norm_shrink(const Dims &dm, const float *part, int splits, size_t slice, const void *resid, void *xsum,
                                  const void *wn, void *y, int R, int K, const void *A0, const void *A1, const RowMeta &rm,
                                  void *T, hipStream_t st);
// the shrink alone, of x [R, K] (row stride ldx)
hipError_t launch_row_shrink(const Dims &dm, const void *x, int ldx, int R, int K, const void *A0, const RowMeta &rm, void *T,
                             hipStream_t st);

bool attn_decode_mfma_supported(const Dims &dm, int g_max);
// Merge of the attention partials of cut sequences (as launch_attn_merge) and, with A0, the shrink of the O projection
// on the merged rows, in one kernel: attn [R][Hq*D] is completed in place, T as for launch_row_shrink.
hipError_t launch_merge_shrink(const Dims &dm, const float *part_o, const float *part_ml, const struct AttnPlan &pl,
                               const int32_t *row_pseq, void *attn, int R, const void *A0, const RowMeta &rm, void *T,
                               hipStream_t st);
// Causal attention of prefill chunks: each plan sequence is a group of consecutive chunk tokens with at
// most attn_prefill_group_queries() stacked queries (tokens x Hq/Hkv).  Whole walks write `out`, pieces of cut ones
// part_o / part_ml (as launch_attn_decode_mfma).
int attn_prefill_group_queries();
int attn_prefill_max_ctx();  // longest piece, in tokens
int attn_prefill_round();    // tokens of a round of the walk: pieces are cut between rounds
// A call goes to the kernel for long pieces: its longest piece, its stacked queries per kv-head, their groups.
bool attn_prefill_pipelined(int longest, int64_t queries, int64_t groups);
bool attn_prefill_mfma_supported(const Dims &dm, int g_max);
hipError_t launch_attn_prefill_mfma(const Dims &dm, const void *q, const void *pool, const int32_t *bt, int max_blocks,
                                    const AttnPlan &pl, void *out, float *part_o, float *part_ml, hipStream_t st);
// part_o: fp32 [slots, Hkv, g_max, D]; part_ml: fp32 [slots, Hkv, g_max, 2] (max in log2 units, sum)
hipError_t launch_attn_decode_mfma(const Dims &dm, const void *q, const void *pool, const int32_t *bt, int max_blocks,
                                   const AttnPlan &pl, void *out, float *part_o, float *part_ml, hipStream_t st);
// row_pseq: plan sequence of each of the R rows; or null: n_seq plan sequences of at most R rows
hipError_t launch_attn_merge(const Dims &dm, const float *part_o, const float *part_ml, const AttnPlan &pl,
                             const int32_t *row_pseq, void *out, int R, int n_seq, hipStream_t st);

// ---- layer stack helpers (index work) ----------------------------------------------------------
// x[row, :] = embed[tok[idx ? idx[row] : row], :]   (rows of row_bytes bytes, a multiple of 16)
hipError_t launch_embed_rows(const void *embed, const int32_t *tok, const int32_t *idx, void *x, int R, int row_bytes, hipStream_t st);
// out[i, :] = x[rows[i], :], and out2[i, :] = x2[rows[i], :] if there is an x2
hipError_t launch_gather_rows(const void *x, const int32_t *rows, void *out, int n, int row_bytes, hipStream_t st, const void *x2 = nullptr,
                              void *out2 = nullptr, int row_bytes2 = 0);
// token[row] = first index of the largest of logits[row, 0..V)
// scratch: argmax_scratch_bytes(R) bytes of device memory, 8-byte aligned (partial results)
size_t argmax_scratch_bytes(int R);
hipError_t launch_argmax(const float *logits, int R, int V, int32_t *token, void *scratch, hipStream_t st);
// seq_next[s] = row_next[last_row[s]]
hipError_t launch_pick_rows(const int32_t *row_next, const int32_t *last_row, int32_t *seq_next, int S, hipStream_t st);

}  // namespace icarus
