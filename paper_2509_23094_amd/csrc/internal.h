// Host-side launch interface between the C ABI layer and the kernel files.
// Every launcher checks its own shape assumptions and returns hipError_t.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace d2c {

enum DType { kF32 = 0, kBF16 = 1 };

inline size_t dtype_size(int dt) { return dt == kBF16 ? 2 : 4; }

// Launch-shape tunables.  Every context holds its own copy (defaults chosen by measurement); the tooling
// calls d2c_init_tuned / d2c_ctx_set_tunable change them per context.
struct Tunables {
  int gemm_target_wgs = 384;   // aim for at least this many groups of 4 waves per GEMM
  int gemm_max_splits = 8;
  int gemm_wide_min_rows = 257; // these from this many rows on (fewer: see the end of plan_gemm)
  int gemm_tall_chunk = 1;      // 129-192 bf16 rows as ONE row chunk of 10 or 12 row tiles (see plan_gemm)
  int gemm_wide_tiles = 1;     // many bf16 rows, 128 x 64 outputs per wave: 0 = never, 1 = the faster by plan_gemm's estimate,
                               // 2 = gemm_wide_kernel, 3 = gemm_rows_kernel with four column tiles
  int gemm_wide_mt = 0;        // row tiles per row chunk of these: 6, 7, 8; 0 = by shape
  int gemm_nt_big_n = 1 << 30; // N above this uses two column tiles per wave even for few rows (measured slower);
                               // more than 128 rows always do
  int gemm_waves = 0;          // waves per workgroup sharing one activation chunk in LDS: 4, 6, 8, 10; 0 = by shape
  bool gemm_preshuffle = true; // d2c_init keeps pre-tiled copies of the projection matrices (costs their size again)
  int gemm_rot = -1;           // start chunk of a workgroup's k walk = (column block * this) % chunks; -1 = by the row pitch
  int attn_tiled_min_m = 96;   // bf16 attention: from this many query rows on, the LDS-tiled kernels (see attention_is_tiled)
  int attn_max_splits = 8;     // key-range splits of one attention launch (1..8)
  int attn_qt = 0;             // 16-row query tiles per wave in the tiled forward kernel: 1, 2; 0 = by m
  int attn_waves = 0;          // waves per workgroup of the tiled forward kernel: 4, 8; 0 = by the time model of plan_fwd
  int attn_target_wgs = 256;   // compute units of that model; a sequence whose workgroups alone are as many is not split
  bool side_stream = false;    // d2c_step: head average + rollout on a second stream (measured slower: with two
                               // queues in use every launch of the step takes longer than the overlap saves)
};
// name -> field; false for an unknown name
bool set_tunable(Tunables& t, const char* name, int value);

// ---- GEMM on a ragged handful of rows: P[s] = A[m,K] * W[N,K]^T over the k-range of split s
struct GemmPlan {
  int mt;        // 16-row tiles per row chunk (1..8, 10, 12)
  int nt;        // 16-column tiles per wave (1, 2 or 4; wide: 3 or 4)
  int waves;     // waves per workgroup (4, 6, 7, 8 or 10), each owning 16*nt output columns
  int splits;    // k splits (partials to be summed by the consumer)
  int k_per_split;
  int row_chunks;
  int rot;       // multiplier of the per-workgroup start-chunk rotation (0 = none)
  bool tile;     // gemm_tile_kernel (float): 16 rows per workgroup, one row_chunk each, whole contractions in flight
  bool wide;     // gemm_wide_kernel: two row chunks per workgroup, four of its 8 waves on each; else gemm_rows_kernel, one

  int chunks_per_wg() const { return wide ? 2 : 1; }
  int cols_per_wg() const { return 16 * nt * waves / chunks_per_wg(); }
};
// Row counts of one tile count (16 t - 15 .. 16 t) on one side of gemm_wide_min_rows have one plan.
// single_split: one split, and the matrix is the gate/up pair with the gated epilogue.  row_major: W as the caller has it.
GemmPlan plan_gemm(const Tunables& t, int dtype, int m, int N, int K, bool single_split = false, bool row_major = false);
// P must hold plan.splits * split_stride floats; split_stride >= m * ldp.
// pre = W is a pre-tiled copy made by launch_preshuffle (then ldw = 256-byte chunks per row).
hipError_t launch_gemm(int dtype, const GemmPlan& plan, const void* A, int lda, const void* W, int ldw,
                       float* P, int ldp, size_t split_stride, int m, int N, int K, hipStream_t st,
                       bool pre = false);
// Pre-tiled weight copy: 16-row x 256-byte blocks, each stored as the 4 x 1 KB wave loads of the
// projection kernel ([tile][chunk][step][lane][16 B]); rows and row tails are zero-padded.
size_t preshuffled_bytes(int N, int K, int dtype);
// interleave_half = F > 0 (N = 2F, F % 16 == 0): 16-row tiles of the two halves alternate (gate, up, gate, ..).
hipError_t launch_preshuffle(int dtype, const void* W, int ldw, int N, int K, void* dst, hipStream_t st,
                             int interleave_half = 0);
// act[m, F] = T(silu(g) * u) with [g | u] = A W^T, W a pre-tiled interleaved copy of [2F, K]; plan: single split
hipError_t launch_gemm_swiglu(int dtype, const GemmPlan& plan, const void* A, int lda, const void* W, int ldw,
                              void* act, int F, int m, int K, hipStream_t st);

// ---- row-wise kernels
// h[r,:] = emb[tokens[idx[r]],:];  a[r,:] = T(rmsnorm(h[r,:]) * gain)
hipError_t launch_embed_norm(int dtype, const void* emb, const int32_t* tokens, const int32_t* idx, int m, int d,
                             const float* gain, float eps, float* h, void* a, hipStream_t st);
// h[r,:] = h_in[r,:] + sum_s P[s][r,:] (n_splits may be 0; then h is not written and h_in is h);
// if a: a[r,:] = T(rmsnorm(h[r,:]) * gain)
hipError_t launch_add_norm(int dtype, const float* h_in, float* h, const float* P, int n_splits, size_t split_stride, int ldp,
                           int m, int d, const float* gain, float eps, void* a, hipStream_t st);
// a[i,:] = T(rmsnorm(h[rows[i],:]) * gain)
hipError_t launch_gather_norm(int dtype, const float* h, const int32_t* rows, int n_rows, int d, const float* gain,
                              float eps, void* a, hipStream_t st);
// split sums of the QKV projection (+bias), RoPE on q and k at the rows' positions; q -> q_out[r,:],
// k -> k_cache[pos,:], v -> v_cache[pos,:].  The compact rows are the concatenation of up to rope_max_batch
// sequences' slices (off = first row of the slice; slices consecutive and non-empty), each with its own
// index set (pos = idx[r - off]) and caches.
struct RopeCall {
  const int32_t* idx;
  void *k_cache, *v_cache;
  int off, m;
};
int rope_max_batch();
// The sequences whose rows one launch covers: rows off .. off+m of the compact buffers belong to a sequence with its own
// index set and caches.
constexpr int kRopeMaxSeqs = 8;
struct RopeSeqs {
  const int32_t* idx[kRopeMaxSeqs];
  void* k_cache[kRopeMaxSeqs];
  void* v_cache[kRopeMaxSeqs];
  int off[kRopeMaxSeqs + 1];          // off[n] = total rows
  int n;
};
__device__ __forceinline__ int rope_seq_of(const RopeSeqs& sq, int r) {
  int s = 0;
  while (s + 1 < sq.n && r >= sq.off[s + 1]) ++s;
  return s;
}
// false: too many, empty or not consecutive
bool rope_seqs(const RopeCall* calls, int n_calls, RopeSeqs& out);
hipError_t launch_qkv_rope_scatter(int dtype, const float* P, int n_splits, size_t split_stride, int ldp,
                                   const float* bias, const RopeCall* calls, int n_calls, int n_heads, int n_kv_heads,
                                   int head_dim, const float* rope_cos, const float* rope_sin, void* q_out,
                                   hipStream_t st);
// What gemm_tile_kernel does beside the product where gemm_fuses (few rows, short contractions, float): the norm (with the
// residual's update) of its activation rows in front, RoPE and the cache update of the QKV projection behind.  Pre-tiled weights.
struct NormFuse {              // A = rmsnorm(h + sum_s P[s]) * gain, [m, K]; h_out (not h itself; null = not wanted) = h + sum_s P[s]
  const float *h, *P;
  int n_splits;
  size_t split_stride;
  int ldp;
  const float* gain;
  float eps;
  float* h_out;
};
struct RopeFuse {              // as launch_qkv_rope_scatter's arguments; 64 must be a multiple of head_dim
  const float* bias;
  const RopeCall* calls;
  int n_calls, n_heads, n_kv_heads, head_dim;
  const float *rope_cos, *rope_sin;
  float* q_out;
};
bool gemm_fuses(int dtype, const GemmPlan& plan);
bool rope_fuses(int head_dim, int n_calls);
// whether the norm that also sums so many splits is the faster inside the projection; qkv_fused: the layer's QKV projection is fused
bool norm_fuses(int n_splits, int K, bool qkv_fused);
// A W^T (norm null: A as given, [m, lda]) turned and written by rope, or (with norm) the gated product to act[m, N / 2]
hipError_t launch_gemm_tile_fused(const GemmPlan& plan, const NormFuse* norm, const float* A, int lda, const void* W, int ldw,
                                  const RopeFuse* rope, float* act, int m, int N, int K, hipStream_t st);
// act[r,f] = T(silu(g) * u), g/u = split sums of columns f and F+f
hipError_t launch_swiglu(int dtype, const float* P, int n_splits, size_t split_stride, int ldp, int m, int F,
                         void* act, hipStream_t st);
// cache_a[idx[r],:] = rows_a[r,:] and, when rows_b is given, cache_b[idx[r],:] = rows_b[r,:].
// Pointers and width*sizeof(T) must be multiples of 16 bytes for the wide path (else element copies).
hipError_t launch_scatter_rows(int dtype, const void* rows_a, void* cache_a, const void* rows_b, void* cache_b,
                               const int32_t* idx, int m, int width, hipStream_t st);
hipError_t launch_copy_f32(float* dst, const float* src, size_t n, hipStream_t st);
// dst[i] = sum_s P[s*split_stride + i], i < n
hipError_t launch_sum_splits(float* dst, const float* P, int n_splits, size_t split_stride, size_t n, hipStream_t st);
// cos/sin table [max_pos, head_dim/2], angles evaluated in fp64
hipError_t launch_rope_table(float* cos_t, float* sin_t, int max_pos, int head_dim, float theta, hipStream_t st);

// ---- attention of m query rows against all L cached keys, no mask
// Two kernel families.  Few query rows (fp32, or bf16 below attn_tiled_min_m rows): a forward launch and, for
// the head average, either per-head probability rows written by the forward launch itself (probs, see
// attention_fwd_emits_probs) or a second launch (launch_attention_avg) that needs the forward's lse.  Many
// rows in bf16 (attention_is_tiled: attn_tiled_min_m rows, or fewer when the key range is too long
// for the probability rows): K/V blocks staged through LDS, key range split over workgroups; the
// forward launch also leaves what the head average needs, and one finishing launch merges the splits and
// writes the average, so tiled_avg is given to launch_attention_fwd itself.
// fwd: out T [m, H*dh] and the log-sum-exp per (head, row), lse float [H, m]
// scratch: attention_scratch_floats(...) floats, may be null for fp32
bool attention_is_tiled(const Tunables& t, int dtype, int m, int L);
size_t attention_scratch_floats(const Tunables& t, int dtype, int max_m, int max_L, int n_heads, int head_dim);
// probs (optional, only where attention_fwd_emits_probs): bf16 [H, m, L], the normalised attention rows of
// every head, written by the same launch; launch_head_mean turns them into the head average.
bool attention_fwd_emits_probs(const Tunables& t, int dtype, int m, int L);
size_t attention_probs_elems(int dtype, int n_heads, int max_L);       // bf16 elements one (layer, sequence) needs
// tiled_avg: float [m, L] or null; only read where attention_is_tiled (elsewhere it must be null)
hipError_t launch_attention_fwd(const Tunables& t, int dtype, const void* q, const void* k_cache, const void* v_cache, int m, int L,
                                int n_heads, int n_kv_heads, int head_dim, void* out, float* lse, float* scratch,
                                size_t scratch_floats, hipStream_t st, void* probs = nullptr,
                                float* tiled_avg = nullptr);
// abar[l] (at abar + l * abar_layer_stride, [m, L]) = mean over heads of probs[l] (at probs + l * stride, [H, m, L])
hipError_t launch_head_mean(const void* probs, size_t probs_layer_stride, float* abar, size_t abar_layer_stride,
                            int n_layers, int n_heads, int m, int L, hipStream_t st);
// the second launch of the few-row kernels: attn_avg float [m, L] = mean over heads of
// exp(q k / sqrt(dh) - lse); needs fwd's lse.  Not for attention_is_tiled shapes.  roll (optional): the rollout block of the
// first layer as launch_rollout's, (attn_avg + one-hot at idx) / 2
hipError_t launch_attention_avg(const Tunables& t, int dtype, const void* q, const void* k_cache, const float* lse, int m, int L,
                                int n_heads, int n_kv_heads, int head_dim, float* attn_avg, hipStream_t st, float* roll = nullptr,
                                const int32_t* idx = nullptr);

// the bf16 kernels for many query rows: forward over a split key range, then one launch that merges the
// splits and (attn_avg != null) writes the head average.  Several sequences (up to attention_tiled_max_batch)
// share the two launches: together they fill the chip with fewer key splits, i.e. fewer partials to merge.
// The scratch is cut into one piece per sequence: it must hold the sum of their needs.
struct TiledCall {
  const void *q, *k_cache, *v_cache;
  int m, L;
  void* out;          // T [m, H*dh]
  float* lse;         // [H, m]
  float* attn_avg;    // [m, L] or null
};
int attention_tiled_max_batch();
size_t attention_tiled_scratch_floats(const Tunables& t, int max_m, int max_L, int n_heads, int head_dim);
hipError_t launch_attention_tiled(const Tunables& t, const TiledCall* calls, int n_calls, int n_heads, int n_kv_heads,
                                  int head_dim, float* scratch, size_t scratch_floats, hipStream_t st);

// ---- rollout on the compact block: c <- (A[:,S] c + A[:,notS] + c) / 2; first: c before is one-hot rows (not read).
// Where rollout_in_place the result replaces c_block, elsewhere it is left in scratch (rollout_scratch_floats(m) and
// at least m * L floats) and the caller copies it back.
bool rollout_in_place(int layer, int m);
size_t rollout_scratch_floats(int max_m);
hipError_t launch_rollout(const float* attn_avg, float* c_block, float* scratch, const int32_t* idx, int m, int L,
                          bool first, hipStream_t st);
hipError_t launch_influence(const float* c_block, const int32_t* idx, int m, int L, float* influence,
                            hipStream_t st);

// ---- Eq. 9 as a row-vector chain: c = 1^T W^(n_layers) ... W^(1) with W^(l) built from abar_l (Eq. 6-7),
// for up to chain_max_batch() independent sequences at once.  abar: layer l of a sequence at abar + l *
// layer_stride, [m, L] floats.  u_scratch: n_layers * (sum of m) floats, g_scratch: n_layers * (sum of m * m)
// floats.  Three launches (the m x m blocks made dense, the sequential m x m part in one workgroup per
// sequence, then all columns in parallel); L <= the selection kernel's limit.
// m == 0 or n_layers == 0: all ones.
struct ChainCall {
  const float* abar;
  const int32_t* idx;
  int m, L;
  float* influence;
};
int chain_max_batch();
hipError_t launch_influence_chain(const ChainCall* calls, int n_calls, size_t layer_stride, int n_layers,
                                  float* u_scratch, float* g_scratch, hipStream_t st);

// ---- selection
// Eq. 1 in two parts: per logits row and chunk of the vocabulary (max, argmax, sum of exp), confidence_chunks(vocab)
// triples per row in part; launch_select merges the rows' chunks into conf and pred before it selects.
// part: confidence_scratch_floats(n_rows, vocab) floats
int confidence_chunks(int vocab);                       // 1..64
size_t confidence_scratch_floats(size_t n_rows, int vocab);
struct SelectArgs {
  float sigma; int k; float p; int block_len; int n_unmask; int cand_mode; float threshold; int conf_decode;
  int32_t* tokens; uint8_t* is_masked; int L; int prompt_len;
  float* conf; int32_t* pred; const float* influence;
  int32_t *mstar, *u_set, *decode_idx, *s_next, *s_rows_next, *counts;
  float* score_out;   // nullable: D(i) * s^i of the stage-1 candidates, 0 elsewhere
  // logit rows of this call whose chunks are still to be merged (n_rows may be 0); a row's position is
  // via ? via[pos[row]] : pos[row].  pos and via may be the s_rows_next / s_next that the call overwrites.
  const float* part; const int32_t *pos, *via; int n_rows, n_chunks;
  // result of the selection's half that needs no logits, kSelPreFloats floats, 8-byte aligned: written by the chunks' launch,
  // read by launch_select.  null (for all sequences of a launch): launch_select does that half as well
  void* pre;
};
constexpr size_t kSelPreFloats = 256 + 4096;      // two bitmaps of 64 words, a float per position of the longest sequence
// first: n_first (up to select_max_batch(), or 0) selections with cand_mode 0 whose first half this launch does too (n_rows > 0 then)
hipError_t launch_confidence_chunks(const float* logits, int n_rows, int vocab, float* part, hipStream_t st,
                                    const SelectArgs* first = nullptr, int n_first = 0);
int select_max_len();
// n independent sequences (n <= select_max_batch), one workgroup each
int select_max_batch();
hipError_t launch_select(const SelectArgs* args, int n, hipStream_t st);
hipError_t launch_seq_reset(const uint8_t* is_masked, int L, int32_t* s_idx, int32_t* s_rows, float* conf,
                            int32_t* pred, int32_t* counts, hipStream_t st);

}  // namespace d2c
