// Host-side launch interface of the gfx950 kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

namespace aed {

enum Dtype { kF32 = 0, kBF16 = 1 };
constexpr int kPage = 16;  // tokens per self-attention KV page

// ---------------------------------------------------------------- decode GEMM
// C[M,N] = prologue(A)[M,K] . W[N,K]^T (+bias), then an epilogue.
// PRO_LNS: the LayerNorm is taken around the product instead of being applied to the operand.
// Whoever writes the residual rows x (embedding, EPI_RESID_S) also writes per-row statistics of x; the gain g of the LayerNorm
// is multiplied into the matrix once, when the decoder is created (Wg = W . diag(g), rounded to the storage type).
// float32: the product reads x itself and takes the row's mean mu off in front of the multiplication,
//   W . LN(x) + bias = rstd * (Wg . (x - mu)) + c2,  c2 = W . b + bias.
// bfloat16: they also write the rows' "shadow" x - mu_hat in the
// storage type and fragment order (mu_hat: the row mean before the update, so the shadow has no large common
// offset), and then
//   W . LN(x) + bias = rstd * (Wg . shadow - (mu - mu_hat) * c1) + c2,  c1 = Wg . 1,
// so the product streams half the bytes of the rows and needs no pass over them first, and one shadow
// serves every product that reads the rows.  (In float32 a shadow would cost more than rounding: where the updates of a layer move a
// row's mean, the product's sums carry that offset.  One layer of d_model 256 whose last update moves the rows by 30 of the
// embeddings' standard deviations, relative error of the logits against float64 with a shadow 7.2e-7, this way 3.2e-7; 300 of them
// 6.5e-6 and 1.8e-6.)
enum GemmPro { PRO_T, PRO_LNS };
// EPI_RESID_S: residual update that also writes the statistics and, bfloat16, the shadow of the updated rows.
enum GemmEpi { EPI_QKV, EPI_F32, EPI_RELU_T, EPI_CROSSKV, EPI_RESID_S };

struct GemmArgs {
    const void* A;        // T [M,K] in fragment order (PRO_LNS: the rows; bfloat16: their shadow)
    int n_raw;            // PRO_LNS + EPI_QKV, streaming kernel: columns [n_raw, N) (n_raw = 3 d_model) are not normalised and not
    float* out2;          // part of q/k/v: their bare sums plus raw_bias go to out2, float [M, N - n_raw] row-major.  0: no such columns
    const float* raw_bias;  // [N - n_raw]
    const float* addend;  // PRO_T + EPI_F32, streaming kernel, may be null: float [M,N] row-major added to the result
    const void* W;        // T [N,K] in fragment order (launch_reorder_weight)
    const void* bias;     // T [N] or null
    float ln_eps;
    int M, N, K;
    void* out;            // EPI_RESID_S: float [M,N] fragment order, += ; EPI_F32: float [M,N] row-major;
                          // EPI_RELU_T: T [M,N] fragment order; EPI_QKV: float q [M,d_model] row-major
    // EPI_QKV: columns [d,2d) and [2d,3d) go to the paged self-attention cache of this layer
    void* k_pool;         // T (or E4M3 codes, kv_fp8) [pages][H][16][Dh]
    void* v_pool;
    const int* kv_slot;     // [M] page * 16 + position inside the page that row m's key / value go to, -1: nowhere
                            // (launch_embed / launch_sample_embed leave it: one load per row and layer instead of state, page table, page)
    int n_heads, head_dim, d_model;
    // EPI_CROSSKV: columns [0,d) -> kc, [d,2d) -> vc, layout [H][t_cap][Dh]
    void* kc;
    void* vc;
    long long t_cap;
    const int* out_row_map;  // EPI_CROSSKV, may be null: frame slot that GEMM row m is written to (default m)
    int a_rows;              // rows the A buffer holds (0: only the next multiple of 128 above M is promised)
    // Row statistics of the residual rows: for every row and every 16-column tile, the tile's mean and its sum
    // of squared deviations from that mean, [rows][stat_tiles] (stat_tiles = d_model / 16; a row is 512 contiguous
    // bytes at d_model = 1024, read by 16 lanes).
    const float2* stats_in;  // PRO_LNS: of A's rows
    // (mu_hat_in, ln_c1, mu_hat_out, shadow_out: bfloat16 only)
    const float* mu_hat_in;  // PRO_LNS: [M] the shift the shadow was written with;
                             // EPI_RESID_S: [M] row means before the update = the shift to write the shadow with
    const float* ln_c1;      // PRO_LNS: [N]
    const float* ln_c2;      // PRO_LNS: [N] (takes the place of bias)
    float* mu_hat_out;       // PRO_LNS, may be null: [M] row means of A's rows, for the residual updates that follow
    float2* stats_out;       // EPI_RESID_S: of the updated rows
    void* shadow_out;        // EPI_RESID_S: T [M,N] fragment order
    int stat_tiles;
    int kv_fp8;              // EPI_QKV / EPI_CROSSKV: the caches hold 8-bit E4M3 codes instead of T
    int rms;                 // the normalisation is RMSNorm (no mean subtraction) instead of LayerNorm: PRO_LNS reads the
                             // statistics that way (see fold_norm)
    int w_nt;                // streaming kernel: load W with the non-temporal hint (weights that are not expected to
                             // survive in the caches until the next step anyway, and should not push other data out)
};

// Buffers in fragment order must hold a multiple of 128 rows (rows >= M are read, never written).
// Returns hipSuccess or the launch error.  Requirements (checked by the caller):
// K % 256 == 0, N % 64 == 0.
hipError_t launch_gemm(Dtype dt, GemmPro pro, GemmEpi epi, const GemmArgs& a, hipStream_t s);
// LDS-tiled MFMA GEMM for large M (bf16 only; fragment-order A padded to a multiple of 128 rows, N % 128 == 0)
hipError_t launch_gemm_tiled(GemmEpi epi, const GemmArgs& a, hipStream_t s);
// the same 128 x 128 tile fed by direct-to-LDS loads (bf16, K >= 512); a.ln_c1 != null: PRO_LNS
hipError_t launch_gemm_dma128(GemmEpi epi, const GemmArgs& a, hipStream_t s);
// bf16 cross K/V product with 256 x 256 tiles fed by direct-to-LDS loads; A must hold whole 256-row tiles
hipError_t launch_gemm_dma_crosskv(const GemmArgs& a, hipStream_t s);
// dst (fragment order [M,K]) <- rows of a row-major source; row m comes from src row row_map[m] (or m); K % 64 == 0
hipError_t launch_reorder_rows(Dtype dt, const void* src, const int* row_map, void* dst, int M, int K, hipStream_t s);
// c1[n] = sum_k T(W[n,k] g[k]) (the column-scaled matrix as it is stored), c2[n] = sum_k W[n,k] b[k] + bias[n]
// (float32 sums; W row-major [N,K]; b and bias may be null)
hipError_t launch_fold_ln(Dtype dt, const void* W, const void* g, const void* b, const void* bias, float* c1, float* c2,
                          int N, int K, hipStream_t s);
// dst (fragment order) <- src (row-major [N,K]), each column k multiplied by gain[k] if gain is given (T [K];
// the product is rounded to T once); N % 16 == 0, K % 64 == 0.  With dst_K > 0 the destination is a fragment-order
// matrix of dst_K columns and src lands in its columns dst_k0 .. dst_k0 + K.
hipError_t launch_reorder_weight(Dtype dt, const void* src, const void* gain, void* dst, int N, int K, hipStream_t s,
                                 int dst_k0 = 0, int dst_K = 0);

// Merged products (bfloat16, at most 256 rows).  A residual update x' = x + Wa . o + ba followed by a LayerNorm
// product Wb . LN(x') reads, in folded form, Wbg . (x' - mu_hat) = Wbg . (x - mu_hat) + (Wbg . Wa) . o + Wbg . ba.
// With the matrix product Wbg . Wa formed once at create, the second product no longer waits for the update:
//   P1 = Wbg . (x - mu_hat) + cb   needs only the shadow of x: computed by the launch that already reads that shadow
//                             (the QKV product, as extra columns: GemmArgs::n_raw, raw_bias),
//   P2 = (Wbg . Wa) . o       needs only o: computed in the same launch as the update (launch_gemm_pair), which
//                             adds P1 to it (GemmArgs::addend),
// and whoever reads P = P1 + P2 finishes it with the statistics of x' that the update's tiles wrote:
//   Wb . LN(x') + bb = rstd' * (P - (mu' - mu_hat) * c1) + c2,  cb = Wbg . ba, c1 = Wbg . 1, c2 = Wb . beta + bb.
// One launch per layer less (self-attention output projection + cross-attention query product).
// launch_gemm_pair: a0 = the update (EPI_RESID_S), a1 = the product P2 (PRO_T, epilogue epi1 = EPI_F32).
hipError_t launch_gemm_pair(Dtype dt, const GemmArgs& a0, GemmEpi epi1, const GemmArgs& a1, hipStream_t s);
// P[n,k] = sum_j T(W1[n,j] g[j]) W2[j,k] -> T, fragment order, columns dst_k0.. of a matrix with dst_K columns
// (W1 [N,J], W2 [J,K] row-major, g null or T [J]; N, K % 64 == 0, J % 16 == 0); bfloat16 only
hipError_t launch_weight_product(Dtype dt, const void* W1, const void* g, const void* W2, void* dst, int N, int J, int K,
                                 int dst_k0, int dst_K, hipStream_t s);
// out[n] = sum_j T(W[n,j] g[j]) v[j] (v null: zeros); bfloat16 only
hipError_t launch_fold_vec(Dtype dt, const void* W, const void* g, const void* v, float* out, int N, int J, hipStream_t s);

// ---------------------------------------------------------------- decode attention
constexpr int kMaxChunks = 8;      // chunks per (sequence, head)
constexpr int kLongItem = 192;     // cross-attention items of that many keys on average are long ones (attn_wavefronts)
constexpr int kItemOff = INT_MIN;  // sign bit of a cross-attention work item's sequence: it has finished
struct AttnArgs {
    const float* q;       // [B, d_model]
    void* out;            // T [B, d_model] in fragment order
    const void* K;        // self: T [pages][H][16][Dh]; cross: T [H][t_cap][Dh]  (this layer)
    const void* V;
    int kv_fp8;           // K and V hold 8-bit E4M3 codes instead of T (bfloat16 mode only)
    // self
    const int* finished;  // [B]
    const int* page_table;
    int max_pages;
    const int* seq_len;   // keys = seq_len[b] + 1
    int chunk;            // keys per work item but a sequence's last, a multiple of 64
    int n_chunks_max;     // grid.z
    int wavefronts;       // per workgroup, self and cross: 4 or 8 (attn_wavefronts)
    int batch;
    // cross
    const int4* items;    // {b (| kItemOff: nothing to do), key_start | chunk_idx << 16, n_keys | n_chunks << 16, first frame of b in the
                          // packed layout}, sequences of several chunks first, then longest first
    int n_items;
    long long t_cap;
    // split-K merge
    float* part;          // [B*H][max_chunks][Dh+2]
    int* counters;        // [B*H] arrivals per (sequence, head); zero between launches
    int max_chunks;
    int n_heads, head_dim;
    float scale_log2e;    // log2(e) / sqrt(Dh)
    // cross-attention behind merged products (see "merged products" above): q holds P, and the kernel finishes it
    // with the statistics of the updated rows: q = rstd' (P - (mu' - mu_hat) c1) + c2.  q_stats null: q is final.
    const float2* q_stats;  // [B][q_stat_tiles] tile statistics of the updated rows
    const float* q_mu_hat;  // [B] shift of the shadow that P was computed from
    const float* q_c1;      // [d_model]
    const float* q_c2;
    float q_eps;
    int q_stat_tiles, q_rms;
};
hipError_t launch_attn_self(Dtype dt, const AttnArgs& a, hipStream_t s);
hipError_t launch_attn_cross(Dtype dt, const AttnArgs& a, hipStream_t s);

// Cross-attention over the encoder frames themselves (attn_frames.hip): bfloat16, d_model 1024, 8 heads of 128
constexpr int kFramesPart = 4;  // positions of a prompt pass that have their queries and sums in the scratch at a time
struct FramesArgs {
    const float* q;       // [rows, 1024]
    const void* wk_t;     // this layer's Wk^T (launch_frames_weight)
    const void* wv;       // rows [1024, 2048) of w_ckv in fragment order
    const void* bv;       // [1024] or null
    const void* frames;   // [.., 1024] in fragment order
    void* q_frames;       // [rows of kFramesPart positions][16][1024] scratch
    void* u_frames;       // the same
    void* out;            // [rows, 1024] in fragment order
    const int4* items;    // AttnArgs::items, whole sequences
    int n_items, rows;
    int positions;        // items i * positions .. + positions - 1 are positions of one sequence, row q * (rows / positions) + b is
                          // position q of sequence b, rows / positions a multiple of 16 (a prompt pass; else 1)
    float scale_log2e;
};
hipError_t launch_attn_frames(const FramesArgs& a, hipStream_t s);
// dst (2 MB): W [1024, 1024] row-major, transposed per head for launch_attn_frames
hipError_t launch_frames_weight(const void* W, void* dst, hipStream_t s);

// ---------------------------------------------------------------- small kernels
struct StateArgs {
    int* seq_len; int* n_gen; int* finished; int* cur_tok; int* limit; int* n_finished;
    int* prompt;      // [B, prompt_stride]
    int* out_tokens;  // [B, out_stride]
    const int* page_table;  // [B][max_pages]
    int* kv_slot;     // [B] see GemmArgs::kv_slot
    int max_pages;
    int prompt_len, prompt_stride, out_stride, max_new;
    int eos_id, pad_id, batch, vocab;
    int4* items;      // [n_items] cross-attention work list (AttnArgs::items): the sampler marks a finished sequence's
    int n_items;      // items with kItemOff, launch_reset and launch_prepare_timing take the marks off
};
// What the LayerNorm of the first layer needs beside the rows themselves (see PRO_LNS).
struct ShadowArgs {
    float2* stats;      // [B][d / 16]: mean and sum of squared deviations of every 16-column tile
    void* shadow;       // bfloat16: T [B, d] fragment order: x - row mean
    float* mu_hat;      // bfloat16: [B] row means (the shadow's shift)
    int rms;            // bfloat16: RMSNorm: the shift is 0 (the shadow is x itself in the storage type)
};
struct EmbedArgs {
    float* x;  // [B, d] fragment order
    const void *tok_emb, *pos_emb;
    int d, max_positions;  // d <= 1024
    float emb_scale;
    ShadowArgs sh;
};
// x[b,:] = emb_scale * tok_emb[cur_tok[b]] + pos_emb[seq_len[b]];  kv_slot[b] = where this step's key / value of
// sequence b go
hipError_t launch_embed(Dtype dt, const EmbedArgs& ea, const StateArgs& st, hipStream_t s);
// a step's end: the argmax, fed next and -> step_out (may be null); every sequence advances
hipError_t launch_sample(const float* logits, const StateArgs& st, int* step_out, hipStream_t s);
// a greedy step's end: prompt feeding, argmax, EOS rules, output writes, then launch_embed of the state that this leaves
hipError_t launch_sample_embed(Dtype dt, const float* logits, const StateArgs& st, const EmbedArgs& ea, hipStream_t s);
// seq_len = start_pos, cur_tok = prompt[b][start_pos], n_gen = finished = 0, n_finished = 0,
// limit = limits ? limits[b] : INT_MAX, out_tokens = pad
hipError_t launch_reset(const StateArgs& st, const int* limits_dev, int start_pos, hipStream_t s);
// The start of a batch: items = src_items (state: n_items of them), counters = 0, state as launch_reset leaves it at position 0 without
// a prompt; with row_map: row_map[src_off[b] + t] = b * t_max + t, where the frames of a padded tensor are.
struct StartArgs {
    const int* src_off;     // [batch + 1] frame offsets, pinned host memory
    const int4* src_items;  // pinned host memory
    int *counters, *row_map;
    int n_counters, t_max;
};
hipError_t launch_start_batch(const StartArgs& a, const StateArgs& st, hipStream_t s);
// ids_out[b] = ids[b], logits_out[i] = logits[i] (i < n, n % 4 == 0); either output may be null, logits_out 16-byte aligned
hipError_t launch_hand_out(const int* ids, int* ids_out, int batch, const float* logits, float* logits_out, size_t n, hipStream_t s);
// cur_tok[b] = src[b * stride]
hipError_t launch_set_tokens(int* cur_tok, const int* src, int stride, int batch, hipStream_t s);
// out[b] = n_gen[b]; dst[b, t] = out_tokens[b, t]
hipError_t launch_copy_out(const StateArgs& st, int* dst_tokens, int* dst_lens, hipStream_t s);

// Slot turnover of the request queue, one workgroup per entry i: slot slots[i] hands its finished request
// old_reqs[i] over (tokens up to n_gen, then pad_id, and the length, into row old_reqs[i] of dst_tokens
// [n_requests, max_new] / dst_lens; -1: nothing to hand over) and starts request new_reqs[i] at position 0 with
// its prompt row of all_prompts [n_requests, prompt_len] and the limit limits[i] (-1: the slot is parked as
// finished).
hipError_t launch_turn_over_slots(const StateArgs& st, const int* slots, const int* old_reqs, const int* new_reqs,
                                  const int* limits, int n, const int* all_prompts, int* dst_tokens, int* dst_lens,
                                  hipStream_t s);

// page_table[b * max_pages + blk] = first_page + b for b < batch (the step API hands every sequence a new page at once)
hipError_t launch_assign_pages(int* page_table, int max_pages, int blk, int first_page, int batch, hipStream_t s);
// p[0 .. n) = 0
hipError_t launch_fill_zero(int* p, int n, hipStream_t s);

// finished[b] = 0, seq_len[b] = clamp(seq_len[b], 0, max_pos), kv_slot to match: a valid mid-decode state for timing runs
hipError_t launch_prepare_timing(const StateArgs& st, int max_pos, hipStream_t s);

}  // namespace aed
