// Host-side launchers of the engine's kernels (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "he_common.h"

enum { EPI_STORE = 0, EPI_BIAS_RELU = 1, EPI_QKV = 2, EPI_STORE_LN = 3, EPI_RESID = 4 };

// ---- plain kernels (kernels_plain.hip): float activations, row-major; bf16 != 0 selects bf16 storage
void plain_embed(hipStream_t s, int bf16, const int32_t* ids, int id_stride, const void* tok, const void* pos, float* x,
                 he_dev_state* st, int M, int S, int H, int V, int pos_offset, const he_step_sampling& sp);
// LayerNorm of rows m*in_mul + in_add of the residual stream
struct plain_ln_args { const void *gamma, *beta; float eps; int in_mul, in_add; };
void plain_ln(hipStream_t s, int bf16, const float* r, const plain_ln_args& ln, float* a, int rows, int H);
// epi: EPI_STORE, EPI_BIAS_RELU, EPI_QKV, or EPI_RESID (out += the product + bias).  ln: A is the residual stream, normalised on
// the way in (scratch [M][K] is used when there are many rows)
void plain_gemm(hipStream_t s, int bf16, const float* A, const void* W, const void* bias, int M, int N, int K, int epi,
                float* out, void* kv, const he_dev_state* st, int S, int layer, int H, int n_heads, int max_batch,
                int max_seq, float qscale, const plain_ln_args* ln = nullptr, float* scratch = nullptr);
int plain_gemm_form(int M, int N, int K);  // HE_PLAIN_ in he.h, of a product that is a launch of its own
void plain_attn(hipStream_t s, int bf16, const float* q, const void* kv, float* o, const he_dev_state* st, int M, int S,
                int layer, int H, int n_heads, int max_batch, int max_seq);
// ---- decode steps of small float models (kernels_blocks.hip): a launch per attention block and per FFN block
struct plain_block_args {
    // the rows: x + pbias + n_part partial sums (attention block of layer 0: embeddings), and the LayerNorm they go through
    const float* pbias; const float *gamma, *beta; float eps; int n_part;
    float* x_out;     // the rows themselves (the LM head: nowhere)
    float* part_out;  // attention block: [n_heads][B][H], FFN block: [F / 32][B][H]
    int H, n_heads, layer, max_batch, max_seq, V;
    const float* bqkv; float qscale;
    const int32_t* ids; int id_stride; const float *tok, *pos; int pos_offset;
    he_step_sampling sp;
};
bool plain_blocks_fit(int B, int H, int n_heads, int F, size_t part_heads, size_t part_slices);
void plain_attn_block(hipStream_t s, bool embed, const float* wqkv, const float* wo, const float* x, const float* part, float* kv, he_dev_state* st,
                      int B, const plain_block_args& a);
int plain_ffn_slices(int F);
void plain_ffn_block(hipStream_t s, const float* w1, const float* w2, const float* x, const float* part, const float* b1, int B, int F,
                     const plain_block_args& a);
void plain_head_block(hipStream_t s, const float* w, const float* x, const float* part, float* logits, int B, const plain_block_args& a);
// rows row0 .. row0+n-1 of the M = B*S positions, given their logits [n][V]: out[b][t] = log_softmax(z)[ids[m+1]]
void plain_score_rows(hipStream_t s, const float* logits, const int32_t* ids, int row0, int n, int S, int V, float* out);

// ---- shared small kernels
// advance > 0: the pass fed that many tokens per sequence and ends here (else launch_advance_state follows)
void launch_sample(hipStream_t s, const float* logits, int B, int V, he_dev_state* st, int32_t* ids_out,
                   float* lp_out, int out_stride, int out_at_step, int32_t* cur_ids, int advance);
// empty cache, greedy sampling, n_counters arrival counters cleared
void launch_reset_state(hipStream_t s, he_dev_state* st, int* counters, int n_counters);
void launch_advance_state(hipStream_t s, he_dev_state* st, int tokens, int steps);
void launch_init_state(hipStream_t s, he_dev_state* st, int max_batch);
// sequences of different lengths: B left-padded rows of S entries, lens[b] of them tokens
void launch_set_ragged(hipStream_t s, he_dev_state* st, const int32_t* lens, int B, int S, int eos_id, int pad_id);
void launch_ragged_post(hipStream_t s, he_dev_state* st, int32_t* gen_ids, float* gen_lp, int32_t* cur_ids, int G, int B);
void launch_fill_gen(hipStream_t s, int32_t* ids, float* lp, int count, const he_dev_state* st);
// Drops the rows of sequences that have ended from the row -> sequence map of the decode steps (`rows` rows so far;
// afterwards as many as sequences are running), and the map back to one row per sequence.
void launch_compact_rows(hipStream_t s, he_dev_state* st, int rows);
void launch_identity_rows(hipStream_t s, he_dev_state* st);
void launch_copy_lens(hipStream_t s, const he_dev_state* st, int32_t* out, int B);
void launch_rng_words(hipStream_t s, uint64_t seed, uint32_t b, uint32_t n, uint32_t v0, int count, uint32_t* out);
void launch_calibration_copy(hipStream_t s, const void* src, void* dst, size_t bytes);
void launch_copy_out(hipStream_t s, const int32_t* ids, const float* lp, int32_t* out_ids, float* out_lp, int count);

// ---- bf16 path (bf16_*.hip): matrix-core operands are tiled blocks of IEEE halves, see bf16_common.h
struct bf16_gemm_args {
    const void* bias = nullptr;      // bf16 [N]
    float* out = nullptr;            // EPI_STORE: partials [ksplit][M][N]; EPI_QKV: q [M][H]
    size_t out_split = 0;            // elements between k-splits
    size_t out_capacity = 0;         // EPI_STORE_LN: floats `out` can hold (0 = not checked)
    void* out_blocks = nullptr;      // EPI_BIAS_RELU: tiled half output
    void* kv = nullptr;              // EPI_QKV
    const he_dev_state* st = nullptr;
    int S = 1, layer = 0, H = 0, n_heads = 0, max_batch = 0, max_seq = 0;
    float qscale = 1.f;
    // LayerNorm folded into the GEMM that consumes it (EPI_BIAS_RELU, EPI_QKV, LM head; decode rows):
    // the activations are gamma * x and ln_stats holds per-column-group statistics of x
    const float* ln_stats = nullptr;  // [m_tiles][ln_groups][32][2] (+ 1 KiB of padding); null = not folded
    int ln_groups = 0, ln_gw = 0, ln_cols = 0;
    float ln_eps = 0.f;
    const float* c1 = nullptr;        // [N padded to 32] W gamma
    const float* c2 = nullptr;        // [N padded to 32] W beta
    // EPI_STORE_LN: k-split sum + bias + residual, gamma * x blocks (out_blocks) and statistics
    float* resid = nullptr;           // [M][N]
    const void* gamma = nullptr;      // bf16 [N] (the caller's parameter)
    float* stats_out = nullptr;       // [m_tiles][groups][32][2]
    int* counters = nullptr;          // [groups * m_tiles] zeros
    // 8-bit weights (bf16_gemm_skinny only): Wp holds E4M3 codes in 16-row units, wscale [N] the row scales 2^e
    const float* wscale = nullptr;
};
// The weights of an EPI_STORE_LN launch by the workgroups that read them, for the launch ahead of it to have them fetched into
// the L2 caches (bf16_attn).  wgs 0: not worth it
struct bf16_ahead {
    const void* w = nullptr;
    int wgs = 0, ks = 1, units = 1, n_units = 0, waves = 8, kbase = 0, kmore = 0, kb = 0, w8 = 0;  // as that kernel is launched
};
// workgroup j's share: units of column group grp, steps k0 .. k0 + n - 1 of k, in lines of 128 bytes; where line l of it lies
struct bf16_ahead_share { int grp, k0, n, lines; };
__host__ __device__ inline bf16_ahead_share bf16_ahead_of(const bf16_ahead& a, int j) {
    const int grp = j / a.ks, p0 = (j - grp * a.ks) * a.waves, p1 = p0 + a.waves;
    const int k0 = p0 * a.kbase + (p0 < a.kmore ? p0 : a.kmore), n = p1 * a.kbase + (p1 < a.kmore ? p1 : a.kmore) - k0;
    return {grp, k0, n, a.units * n * 8};
}
__host__ __device__ inline size_t bf16_ahead_line(const bf16_ahead& a, const bf16_ahead_share& s, int l) {
    const int q = l & 7, i = l >> 3, t = i / s.n, step = s.k0 + i - t * s.n;
    const int u = s.grp * a.units + t, g = u < a.n_units - 1 ? u : a.n_units - 1;  // (past the last unit: it again)
    return a.w8 ? ((size_t)g * (a.kb / 4) + step) * 1024 + q * 128
                : (size_t)(g >> 1) * a.kb * 1024 + (size_t)step * 2048 + (q >> 1) * 512 + (g & 1) * 256 + (q & 1) * 128;
}
bf16_ahead bf16_store_ahead(const void* Wp, int M, int N, int K, size_t capacity, bool w8);
size_t bf16_tiled_bytes(int rows, int K);
void bf16_tile_rows(hipStream_t s, const void* src, void* dst, int R, int K);
// dst = tiled bf16(src + scale * B A): A bf16 [rank, K], B bf16 [R, rank]
void bf16_tile_rows_lora(hipStream_t s, const void* src, void* dst, int R, int K, const void* A, const void* B, int rank,
                         float scale);
// The same (A null: without an adapter; src null: dst holds the tiles already), and c1 = W gamma, c2 = W beta of the R rows padded to 32
void bf16_tile_fold(hipStream_t s, const void* src, void* dst, int R, int K, const void* A, const void* B, int rank, float scale,
                    const void* gamma, const void* beta, float* c1, float* c2);
// EPI_STORE_LN GEMM of M <= 64 rows: columns per workgroup (= per group of LayerNorm statistics) and k-splits;
// capacity = floats of k-split scratch available (the value passed as bf16_gemm_args.out_capacity); w8 != 0: 8-bit weights
void bf16_store_plan(int M, int N, int K, size_t capacity, int w8, int* group_cols, int* ks);
// floats of k-split scratch that launch may index (upper bound); w8 != 0: the 8-bit-weight plan
size_t bf16_store_need(int M, int N, int K, size_t capacity, int w8);
// What that launch indexes, from the launcher's own choice of kernel variant and grid (host logic, no launch).
// cus: compute units to plan for (0 = the current device's).  need_floats: what bf16_store_need answers.
void bf16_store_footprint(int M, int N, int K, size_t capacity, int w8, int cus, size_t* scratch_floats,
                          size_t* need_floats, int* cells, int* stat_groups, int* ksplit);
// the launch plan itself (host logic only; cus > 0 overrides the device's CU count): rows per unit (32 or 16),
// units per workgroup, k-splits; store != 0 for the k-split GEMMs
void bf16_plan_query(int M, int N, int K, int store, size_t capacity, int cus, int* unit_rows, int* per_wg, int* ks);
void bf16_embed_ln(hipStream_t s, const int32_t* ids, int id_stride, const void* tok, const void* pos,
                   he_dev_state* st, int B, int H, int V, int pos_offset, int gw, const void* gamma, float* r,
                   void* x_blocks, float* stats, const he_step_sampling& sp);
// rows b*S + S-1 of r and q ([B*S][H] floats) -> rows b of r_out and q_out ([B][H]); the state advances by `advance` tokens
void bf16_gather_last_rows(hipStream_t s, const float* r, const float* q, float* r_out, float* q_out, int B, int S, int H, he_dev_state* st,
                           int advance);
// rows in slices of 32 (a decode step; 33 to 64 sequences: both slices to a workgroup): EPI_BIAS_RELU, EPI_QKV or EPI_STORE_LN;
// X: the activations as tiled half blocks; ksplit is ignored (the plan decides)
void bf16_gemm_skinny(hipStream_t s, int mode, const void* Wp, const void* X, int M, int N, int K, int ksplit,
                      const bf16_gemm_args& a);
// ... on 8-bit weights: Wp holds E4M3 units, `units` of them to a workgroup
void bf16_gemm_units8(hipStream_t s, int mode, const void* Wp, const void* X, int M, int N, int K, int units, int ksplit,
                      const bf16_gemm_args& a);
// Many rows (prompt and scoring passes, wide decode steps): EPI_BIAS_RELU or EPI_QKV.  part: scratch of part_floats
// floats for the k ranges' sums where the tiles alone do not fill the chip (a second kernel then adds them and applies
// the epilogue).
void bf16_gemm_tiled(hipStream_t s, int mode, const void* Wp, const void* X, int M, int N, int K, const bf16_gemm_args& a,
                     float* part, size_t part_floats);
// The GEMMs whose partial sums the following LayerNorm adds (out-projection, FC2): the plan -- tile shape, *ks k ranges for
// the columns >= *split_col, one for the columns before -- and the launch: part [ks][M][N]
// (few_rows_whole: passes of too few rows for rounds of big tiles get one k range)
void bf16_tiled_store_plan(int M, int N, int K, size_t capacity_floats, int* tile, int* ks, int* split_col,
                           bool few_rows_whole = false);
void bf16_gemm_tiled_store(hipStream_t s, const void* Wp, const void* X, int M, int N, int K, float* part, int tile, int ks,
                           int split_col);
// floats of scratch these can make use of for passes of up to `rows` rows and matrices of up to `widest` rows
size_t bf16_tiled_scratch_floats(int rows, int widest);
// The plan of a many-row GEMM for a planner query (cus: compute units to plan for, 0 = the current device's)
void bf16_tiled_plan_query(int M, int N, int K, int may_cut, size_t capacity_floats, int cus, int* tile_cols, int* ks,
                           int* split_col);
// What the launchers choose for any of these GEMMs (capacity_floats: the scratch they are given): *tile_rows x *tile_cols tiles
// (32 x 32: the LM head streamed in slices of 32 rows), *wg_cols columns of one to a workgroup (128: a halved tile)
enum { TILED_STORE = 0, TILED_STORE_WHOLE = 1, TILED_FUSED = 2, TILED_LM_HEAD = 3, TILED_SCORE_HEAD = 4 };
void bf16_pass_plan_query(int use, int M, int N, int K, size_t capacity_floats, int cus, int* tile_rows, int* tile_cols, int* wg_cols, int* ks,
                          int* split_col);
// whether a launch of the few-row tiles copies its weights past the caches
bool bf16_ring_streams(int M, int N, int K, int tile_rows, int wg_cols, int ksplit);
// ---- 8-bit weight storage: E4M3 codes with one power-of-two scale per row
size_t fp8_units_bytes(int rows, int K);  // codes in the half-tile kernel's units: [rows/16][K/64][64 lanes][16 bytes]
void fp8_row_exponents(hipStream_t s, const void* src, int R, int K, int* exps, float* scales);  // e[n], 2^e[n]
void fp8_quant_rows(hipStream_t s, const void* src, const int* exps, void* codes, int R, int K);  // row-major codes
void fp8_quant_units(hipStream_t s, const void* src, const int* exps, void* units, int R, int K);
// units -> half 32x16 blocks (what the tiled GEMMs read)
void fp8_dequant_units(hipStream_t s, const void* units, const float* scales, void* dst_blocks, int R, int K);
// advance: the step ends here (else launch_advance_state follows)
void bf16_lm_head(hipStream_t s, const void* Wp, const void* X, int B, int V, int K,
                  he_dev_state* st, float* logits_opt, float* stats, int* stats_idx, int32_t* ids_out,
                  float* lp_out, int out_stride, int out_at_step, int32_t* cur_ids, bool advance,
                  const bf16_gemm_args* fold = nullptr);
// partials per row that any form of the LM head leaves, at most
int bf16_lm_parts_max(int V);
// whether it streams the matrix in slices of 32 rows (host logic)
bool bf16_lm_head_streams(int B, int V);
// ... else (bf16_lm_head calls it): soft-max and arg-max partials into stats / stats_idx; returns how many per row
int bf16_lm_head_tiles(hipStream_t s, const void* Wp, const void* X, int M, int V, int K, const bf16_gemm_args* fold, const he_dev_state* st,
                       float* logits_opt, float* stats, int* stats_idx);
// LM head over all M = B*S positions fused with log-softmax and the gather of each position's next
// token: out [B][S-1]; stats [M][bf16_score_parts(V)][2] and tgt [M] are scratch
int bf16_score_parts(int V);
void bf16_score_head(hipStream_t s, const void* Wp, const void* X, int M, int S, int V, int K,
                     const int32_t* ids, float* stats, float* tgt, float* out);
// split_col: with two k ranges, the first column that has the second partial sum (0: every column; a multiple of 256)
void bf16_ln(hipStream_t s, float* r, const float* part, int ksplit, size_t part_split, const void* pbias,
             const void* gamma, const void* beta, void* a_blocks, int rows, int H, float eps, int in_mul, int in_add,
             int writeback, int split_col = 0);
void bf16_attn(hipStream_t s, const float* q, const void* kv, void* o_blocks, const he_dev_state* st, int M, int S,
               int layer, int H, int n_heads, int max_batch, int max_seq, const bf16_ahead* ahead = nullptr);
// host logic: which kernel that launch is (HE_ATTN_ in he.h), wavefronts to a workgroup
void bf16_attn_plan_query(int M, int S, int n_heads, int d, int max_seq, int cus, int* form, int* waves);
