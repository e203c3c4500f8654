// Host-side launchers of the HIP kernels (one translation unit per kernel family).
#pragma once
#include "common.hpp"

namespace sun {

// ---------------- projections (proj.hip) ----------------

enum ProjEpilogue {
    EPI_STORE = 0,   // fp32 partial sums: out[(split * ld_rows + b) * ldo + n]
    EPI_SWIGLU = 1   // gate/up pair, bf16 weights, no split: out is the two-plane tile of silu(gate) * up [rows, N/2]
};

struct ProjLaunch {
    const Mat* W;
    const void* A;         // tiled bf16 activations [rows, K]
    const float* qscale;   // W4 only: [K/128][MB*32] pairs (scale, sum of integers as int bits) of the fixed-point tile A
    int rows;              // valid rows (<= 256; bf16 weights: <= kMaxPrefillTile)
    int epilogue;
    int splits;            // split-K factor (EPI_STORE only); partial s is written at out + s*ld_rows*ldo
    float* out;
    int ldo;               // leading dimension of out (>= N)
    int ld_rows;           // rows per split slab
};
// Chooses the split-K factor the step uses for this matrix and row count.
int proj_pick_splits(const Mat& W, int rows, int max_splits);
bool proj_fuses_swiglu(const Mat& gu, int rows);  // gate/up: one launch with EPI_SWIGLU rather than slabs and launch_swiglu_tile
hipError_t launch_proj(const ProjLaunch& p, hipStream_t st);

// fp32 activations path (vector ALU): y[b][n] = sum_k W[n][k] h[b][k] with h = x, or rmsnorm(x) * gain when gain is given;
// row-major, out[b][n] = y, out[b][n] += y (out is not x), or for a gate/up pair out [rows, N/2] = silu(gate) * up.
enum F32Epilogue { F32_STORE = 0, F32_ADD = 1, F32_SWIGLU = 2 };
bool f32_fuses_norm(const Mat& W, int rows, int epilogue);  // the norm inside the projection rather than in a launch of its own
hipError_t launch_proj_f32(const Mat& W, const float* x, int rows, const void* gain, float eps, int epilogue, float* out, hipStream_t st);

// packing (weights load time)
size_t packed_bf16_bytes(int N, int K);
size_t packed_w4_bytes(int N, int K);     // codes
size_t packed_w4_sz_bytes(int N, int K);  // scales / zero points
// mode 0: rows of up to three sources stacked; mode 1: two sources interleaved in blocks of 16 rows.
hipError_t launch_pack_bf16(const void* const src[3], const int src_rows[3], int nsrc, int mode, int K,
                            void* dst, hipStream_t st);
hipError_t launch_pack_w4(const sun_qmat src[3], const int src_rows[3], int nsrc, int mode, int K,
                          void* dst_codes, void* dst_sz, hipStream_t st);
hipError_t launch_quantize_w4(const void* w, int dtype, int rows, int cols, int group, int mode, void* q,
                              void* s, void* z, hipStream_t st);

// ---------------- attention (attention.hip) ----------------

struct AttnPlan {           // device arrays inside the workspace
    int32_t* chunk_off;     // [batch+1] prefix sum of chunks (full + small) per request
    int32_t* full_off;      // [batch+1] prefix sum of full chunks per request
    int32_t* records;       // [max_chunks * Hkv][24] per-item records
    float* partial;         // [max_chunks][Hq][d+2]  (o[d], m, l)
    int max_chunks;
};
size_t attn_max_chunks(int batch, int max_pages, int Hkv);
hipError_t launch_attn_plan(const AttnPlan& plan, const int32_t* n_or_len, int len_plus, int batch,
                            const int32_t* page_tables, int max_pages, int n_pages, int Hkv, hipStream_t st);
// K in whole token rows past the caches, the same through the caches, or as the operand lies through the caches.
enum KRead { K_STREAMED, K_ROWS, K_IN_PLACE };
// First launch of a decode step: launch_embed_rope and launch_attn_plan (n_tokens = seq_lens + 1) together.
// Counters of the launch that runs all layers, and its word that says it was given up, start at zero.
struct LayersZero {
    uint32_t* p;
    int n;
    uint32_t* lost;
};
hipError_t launch_step_begin(const sun_model_cfg& cfg, const void* embed, const int32_t* tokens, const int32_t* seq_lens, int batch,
                             float* x, float* table, const AttnPlan& plan, const int32_t* page_tables, int max_pages,
                             int n_pages, LayersZero zero, hipStream_t st);
// n_tokens(i) = n_or_len[i] + len_plus.  q fp32 [batch, Hq*d].  The chunk counts of the batch (all chunks, full
// chunks) when the host knows the lengths, else < 0.
hipError_t launch_attn_split(const KvPool& pool, int layer, const AttnPlan& plan, const float* q,
                             const int32_t* page_tables, int max_pages, const int32_t* n_or_len, int len_plus,
                             int batch, int total_chunks_hint, int full_chunks_hint, KRead k_read, bool f32_exact, hipStream_t st);
// How the K of the cached tokens is read (128 dims; the same sums whichever).  W: NULL where attention is all that runs.
KRead attn_k_read(const sun_model_cfg& c, const Weights* W, long long tokens);
// out: fp32 row-major [batch, Hq*d] (out_f32) and/or the O projection's input: two-plane tiled bf16, or, with
// qscale given, the fixed-point tile of a 4-bit projection and its (scale, integer sum) pairs.
hipError_t launch_attn_combine(const sun_model_cfg& cfg, const AttnPlan& plan, int batch, float* out_f32,
                               void* out_tiled, float* qscale, hipStream_t st);

// fp32, tables of at most kShortTokens positions (fewer with many or wide query heads): launch_rope_append, launch_attn_split and launch_attn_combine of a decode step in
// one launch, bit for bit.  qkv [batch, (Hq + 2 Hkv) * d], out [batch, Hq * d].
constexpr int kShortTokens = 384, kShortShare = 1024;   // chunks x query heads of a KV head x dims; measured in attention.hip
bool attn_short_f32(const sun_model_cfg& c, int max_pages);
hipError_t launch_attn_short_f32(const KvPool& pool, int layer, const float* qkv, const float* table, const int32_t* seq_lens, const int32_t* page_tables,
                                 int max_pages, int batch, const LayerW& w, float* out, hipStream_t st);

// Causal attention of `rows` consecutive positions first .. first + rows - 1 of one request over positions 0 .. its own;
// K and V of all of them are in the pool.  q fp32 [rows, Hq*d], rotated; out: two-plane tile of the O projection.
// splits > 1: the keys are split and merged again, partial is scratch of [rows][splits][Hq][d + 2] floats.
hipError_t launch_attn_prefill(const KvPool& pool, int layer, const float* q, const int32_t* page_table, int first, int rows,
                               int splits, float* partial, void* out_tiled, hipStream_t st);
// how many splits the block wants
int attn_prefill_splits(const sun_model_cfg& c, int rows, int first);

// ---------------- all layers of a small batch in one launch (layers.hip) ----------------
constexpr int kLayersRows = 16;    // rows of such a step at most; measured in layers.hip
constexpr int kLayersRowsW4 = 8;   // with 4-bit weights
struct LayersScratch {
    void* p;
    size_t bytes;
};
bool layers_usable(const Weights& W, int rows, const LayersScratch& scratch, hipStream_t st);
// A launch that was given up says so in a word of the plan's first array, behind the prefix sums of so few rows and within the 256 bytes
// that the array's place is rounded up to; it outlives the step's other scratch.
constexpr int kLostAt = 32;
static_assert(kLayersRows + 1 <= kLostAt && kLostAt < 64, "a place of its own");
inline uint32_t* layers_lost(const AttnPlan& plan) { return (uint32_t*)plan.chunk_off + kLostAt; }
LayersZero layers_zero(const LayersScratch& scratch, const Weights& W, const AttnPlan& plan);
// x: the embedding on entry, the residual stream behind the last layer on return, or nothing of use where the launch was given up (after
// `polls` polls of one wait in vain); cache entries that it has appended by then are right.  Behind launch_step_begin with
// layers_zero() of the same scratch.
hipError_t launch_layers(const KvPool& pool, const Weights& W, int rows, float* x, const float* table, const AttnPlan& plan,
                         const int32_t* page_tables, int max_pages, const int32_t* seq_lens, int total_chunks_hint, int full_chunks_hint,
                         const LayersScratch& scratch, unsigned polls, hipStream_t st);

// Workgroups of a kernel (one per compute unit, at most `most`) that a cooperative launch on the device keeps resident; 0: none.
int resident_grid(const void* kernel, int threads, int most, int dev);
bool is_capturing(hipStream_t st);   // or cannot tell
bool has_all_units(hipStream_t st);  // not confined to some of the compute units (false if it cannot tell)

// ---------------- everything else (misc.hip) ----------------

// Embedding rows and rotary tables; position of row b: seq_lens[b], or first_pos + b when seq_lens is NULL.
hipError_t launch_embed_rope(const sun_model_cfg& cfg, const void* embed, const int32_t* tokens, const int32_t* seq_lens,
                             int first_pos, int rows, float* x, float* table, hipStream_t st);
// x[b] += sum_s partial[s][b] (s ascending; nparts may be 0); then h = rmsnorm(x; g).
// h_f32 (fp32 gains): row-major.  Else h_tiled (bf16 gains): two-plane tiled bf16; with qscale given the fixed-point tile of a 4-bit projection instead, and qscale
// receives its (scale, integer sum) pairs.  lost (may be NULL; not with h_f32): where *lost is not 0, h is not-a-numbers.
hipError_t launch_residual_norm(const sun_model_cfg& cfg, float* x, const float* partial, int nparts, int ld_rows,
                                const void* gain, int batch, float* h_f32, void* h_tiled, float* qscale, hipStream_t st,
                                const uint32_t* lost = nullptr);
// k_src, v_src: bf16 [n_layers][n_tokens][Hkv][d]; token t lands at position first_pos + t of the request whose
// page-table row is given.
hipError_t launch_kv_ingest(const KvPool& pool, const void* k_src, const void* v_src, int n_tokens, int first_pos,
                            const int32_t* page_table, hipStream_t st);
// Between two steps of a run: token feedback, length + 1, page allocation in request order.  A request without a token (next < 0)
// stays as it is, status bit 2.
hipError_t launch_advance(const int32_t* next, int batch, int max_pages, const int32_t* free_pages, int n_free,
                          int32_t* token_ids, int32_t* page_tables, int32_t* seq_lens, int32_t* free_head,
                          int32_t* status, bool clear_status, hipStream_t st);
// Between two steps of a run (fp32): launch_argmax, launch_advance and, unless it was the last step, the next step's embedding rows and
// rotary table, in one launch.
constexpr int kTurnRows = 64, kTurnVocab = 1 << 15, kTurnLogits = 1 << 17;   // requests, logits of one and of all of them, at most
hipError_t launch_run_turn(const sun_model_cfg& cfg, const void* embed, const float* logits, int batch, int max_pages, const int32_t* free_pages, int n_free,
                           int32_t* next, int32_t* token_ids, int32_t* page_tables, int32_t* seq_lens, int32_t* free_head, int32_t* status,
                           bool clear_status, bool last, float* x, float* table, hipStream_t st);
// Per-row inputs of one block of a prefill: row r gets a copy of the request's page-table row, length
// first_pos + r and the source-model id.
hipError_t launch_prefill_rows(const int32_t* page_table, int max_pages, int first_pos, int model_id, int rows,
                               int32_t* tables, int32_t* lens, int32_t* ids, hipStream_t st);
// Rows, waiting queue and page ring of a decode worker with continuous batching (sun_serve_state plus sizes).
struct ServeArgs {
    int32_t *token_ids, *page_tables, *seq_lens, *model_ids, *slot_req, *slot_left;
    const int32_t *w_req, *w_token, *w_tables, *w_lens, *w_model, *w_budget;
    int32_t *ring, *counters;
    int n_wait, ring_cap, idle_page, eos_id, slots, max_pages;
};
// Between two steps (advance) and/or before the first (reset): record tokens, retire, grow, admit.
hipError_t launch_serve(const ServeArgs& a, const int32_t* next, int32_t* tokens_out, int32_t* req_out, bool reset,
                        bool advance, hipStream_t st);
// qkv partial sums [nparts][ld_rows][Nqkv] -> rotated q fp32 [batch, Hq*d]; K,V (bf16) appended to the pool.
// seq_lens NULL: row b is position first_pos + b of one request, whose page-table row is page_tables.
hipError_t launch_rope_append(const KvPool& pool, int layer, const float* qkv, int nparts, int ld_rows,
                              const float* table, const int32_t* seq_lens, int first_pos, const int32_t* page_tables, int max_pages,
                              int batch, float* q_out, const void* q_norm, const void* k_norm, const void* bq, const void* bk,
                              const void* bv, hipStream_t st);
// gate/up partial sums (projection column order) -> silu(g)*u as two-plane tiled bf16, or as fixed-point tile + qscale
hipError_t launch_swiglu_tile(const float* part, int nparts, int ld_rows, int rows, int ffn, void* tiled, float* qscale,
                              hipStream_t st);
// measurement only: read n_blocks blocks of block_units 16-byte units (order given by perm, or address order),
// with plain loads or with the streaming loads the attention kernel uses for K and V
hipError_t launch_hbm_read_probe(const void* src, long long n_blocks, int block_units, const int32_t* perm, int grid,
                                 bool stream, uint32_t* sink, hipStream_t st);
constexpr int kArgmaxParts = 16;    // slices of a logits row searched by separate workgroups
constexpr int kArgmaxOne = 4096;    // a row of at most this many logits is searched by one
// part_val / part_idx: scratch [batch][kArgmaxParts].  lost (may be NULL): where *lost is not 0 there are no tokens, next = -1.
hipError_t launch_argmax(const float* logits, int batch, int vocab, float* part_val, int32_t* part_idx, int32_t* next,
                         const uint32_t* lost, hipStream_t st);
// fp32 [rows, K] -> two-plane tiled bf16, or fixed-point tile + qscale
hipError_t launch_tile_rows(const float* x, int rows, int K, void* tiled, float* qscale, hipStream_t st);
// out[b][n] = sum_s partial[s][b][n]
hipError_t launch_reduce_partials(const float* partial, int nparts, int ld_rows, int rows, int N, float* out,
                                  hipStream_t st);
// tiled bf16 [rows, K] -> fp32 row-major
hipError_t launch_untile_rows(const void* tiled, int rows, int K, float* out, hipStream_t st);

}  // namespace sun
