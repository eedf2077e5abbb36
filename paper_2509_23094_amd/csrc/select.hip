// Selection side of the d2Cache step: Eq. 1 (prediction and confidence over the
// vocabulary), Eq. 3-4 (certainty density, stage-1 top-k), unmasking (Eq. 2),
// the rollout update on the compact |S| x L block (Eq. 6-8), influence scores
// (Eq. 9) and the stage-2 cumulative-mass selection (Sec. 4.2, last paragraph).
//
// Everything that decides an index is integer-exact and order-independent:
// top-k ranks keys (float bits of the non-negative score, then lower index
// first); top-p looks for the key at which the fixed-point masses
// floor(c * 2^32), added up in uint64, cross the threshold.  Ties always go to
// the lowest index.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace d2c {
namespace {

typedef unsigned long long u64;
__device__ __forceinline__ u64 low_mask(int n) { return n <= 0 ? 0ull : n >= 64 ? ~0ull : (1ull << n) - 1ull; }

// ------------------------------------------------------------------ Eq. 1
// x-hat = argmax_v, s = 1 / sum_v exp(x_v - max).  A vocabulary row (0.5 MB at V = 126464) is cut into
// chunks, one workgroup each, so that a few dozen rows still fill the chip: per chunk (max, first index of
// the max, sum of exp(x - chunk max)); merge_rows puts the chunks of a row together (ties keep the lowest index) in an
// order that depends on the vocabulary alone -- bit-reproducible, whatever else the call holds.
constexpr int kConfThreads = 256;
constexpr int kConfMaxChunks = 64;
constexpr int kConfChunk = 8192;              // entries per chunk, as long as 64 chunks cover the vocabulary

// One chunk by four waves of a workgroup; the barriers inside are the whole workgroup's, whose waves all have a chunk.
struct ConfLds {
  float val[kConfThreads / 64];
  int idx[kConfThreads / 64];
  float sum[kConfThreads / 64];
};
__device__ __forceinline__ void confidence_chunk(const float* __restrict__ logits, int vocab, int chunk, int n_chunks,
                                                 float* __restrict__ part, int row, int ck, ConfLds& lds) {
  float (&s_val)[kConfThreads / 64] = lds.val;
  int (&s_idx)[kConfThreads / 64] = lds.idx;
  float (&s_sum)[kConfThreads / 64] = lds.sum;
  const float* x = logits + (size_t)row * vocab;
  const int lo = ck * chunk, hi = min(vocab, lo + chunk);
  const int tid = threadIdx.x % kConfThreads, wave = tid >> 6, lane = tid & 63;
  float best = -INFINITY;
  int bidx = 0x7fffffff;
  for (int v = lo + tid; v < hi; v += kConfThreads) {       // ascending per thread: a tie keeps the lower index
    const float xv = x[v];
    if (xv > best) { best = xv; bidx = v; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o, kWave);
    const int oi = __shfl_xor(bidx, o, kWave);
    if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
  }
  if (lane == 0) { s_val[wave] = best; s_idx[wave] = bidx; }
  __syncthreads();
  best = s_val[0]; bidx = s_idx[0];
  for (int w = 1; w < kConfThreads / 64; ++w) {
    const float ob = s_val[w];
    const int oi = s_idx[w];
    if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
  }
  float sum = 0.f;
  for (int v = lo + tid; v < hi; v += kConfThreads) sum += expf(x[v] - best);
  sum = wave_sum(sum);
  if (lane == 0) s_sum[wave] = sum;
  __syncthreads();
  if (tid == 0) {
    float t = 0.f;
    for (int w = 0; w < kConfThreads / 64; ++w) t += s_sum[w];
    float* o = part + ((size_t)row * n_chunks + ck) * 3;
    o[0] = best;
    o[1] = __int_as_float(bidx);
    o[2] = t;
  }
}

// The same for chunks of exactly 8192 entries of 16-byte aligned rows (vocab % 4 == 0): a thread keeps its 32
// entries in registers (eight 16-byte loads issued together), so the row is read once and the kernel is one
// memory latency long.  Entry order per thread is ascending (piece, then element), as the tie rule needs.
__device__ __forceinline__ void confidence_chunk_vec(const float* __restrict__ logits, int vocab, int n_chunks,
                                                     float* __restrict__ part, int row, int ck, ConfLds& lds) {
  constexpr int kChunk = kConfChunk, kPieces = kChunk / (4 * kConfThreads);
  float (&s_val)[kConfThreads / 64] = lds.val;
  int (&s_idx)[kConfThreads / 64] = lds.idx;
  float (&s_sum)[kConfThreads / 64] = lds.sum;
  const float* x = logits + (size_t)row * vocab;
  const int lo = ck * kChunk;
  const int tid = threadIdx.x % kConfThreads, wave = tid >> 6, lane = tid & 63;
  f32x4 val[kPieces];
#pragma unroll
  for (int p = 0; p < kPieces; ++p) {
    const int v = lo + (p * kConfThreads + tid) * 4;
    val[p] = *reinterpret_cast<const f32x4*>(x + min(v, vocab - 4));       // past the end: re-read, masked below
  }
  float best = -INFINITY;
  int bidx = 0x7fffffff;
#pragma unroll
  for (int p = 0; p < kPieces; ++p) {
    const int v = lo + (p * kConfThreads + tid) * 4;
    if (v >= vocab) val[p] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (val[p][e] > best) { best = val[p][e]; bidx = v + e; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o, kWave);
    const int oi = __shfl_xor(bidx, o, kWave);
    if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
  }
  if (lane == 0) { s_val[wave] = best; s_idx[wave] = bidx; }
  __syncthreads();
  best = s_val[0]; bidx = s_idx[0];
  for (int w = 1; w < kConfThreads / 64; ++w) {
    const float ob = s_val[w];
    const int oi = s_idx[w];
    if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
  }
  float sum = 0.f;
#pragma unroll
  for (int p = 0; p < kPieces; ++p)
#pragma unroll
    for (int e = 0; e < 4; ++e) sum += expf(val[p][e] - best);              // exp(-inf) = 0 past the end
  sum = wave_sum(sum);
  if (lane == 0) s_sum[wave] = sum;
  __syncthreads();
  if (tid == 0) {
    float t = 0.f;
    for (int w = 0; w < kConfThreads / 64; ++w) t += s_sum[w];
    float* o = part + ((size_t)row * n_chunks + ck) * 3;
    o[0] = best;
    o[1] = __int_as_float(bidx);
    o[2] = t;
  }
}

// ------------------------------------------------------------------ Eq. 6-8 on the compact block
// c_out[i, c] = ( sum_r A[i, S_r] c_in[r, c] + A[i, c] [c not in S] + c_in[i, c] ) / 2
// Rows outside S stay one-hot under Eq. 6-7, so only these m rows ever change.
constexpr int kRollThreads = 256;

// First layer: C^(0) = I, so sum_r A[i,S_r][c == S_r] + A[i,c][c not in S] = A[i,c] and c_in[i,c] = [c == S_i].
__global__ __launch_bounds__(kRollThreads) void rollout_first_kernel(const float* __restrict__ A,
                                                                     float* __restrict__ c_out,
                                                                     const int32_t* __restrict__ idx, int m, int L) {
  const int col = blockIdx.x * kRollThreads + threadIdx.x;
  const int i = blockIdx.y;
  if (col >= L) return;
  c_out[(size_t)i * L + col] = 0.5f * (A[(size_t)i * L + col] + (idx[i] == col ? 1.f : 0.f));
}

// Later layers: the m x m by m x L product on the fp32 matrix cores, in place.  One workgroup owns 16 columns: it
// keeps its strip of c_in in LDS, so that nobody else reads what it overwrites, and its 8 waves take the 16-row tiles
// round-robin.  Per 16-long step of the contraction a lane holds A[i0 + l%16][S[k0 + 4(l/16) + e]] and
// C[k0 + 4(l/16) + e][c0 + l%16], e = 0..3, one 16x16x4 instruction per e.
// DENSE: the operand A[:, S] comes from a dense copy (16 bytes a lane) instead of being gathered again by each of the
// L / 16 workgroups (64 cache lines a load); it costs a launch, so few rows gather.  Per update, with the launches it
// takes: 97 rows x 1823 columns 12.3 us gathered, 10.4 dense (15.5 with the copy that the tile kernel below needs);
// 37 x 128 5.2 gathered, 6.0 dense; 600 x 3072 169 us in the tile kernel, 69 now; 1024 x 3072 413 -> 152.
constexpr int kRollStripThreads = 512, kRollStripWaves = 8;
constexpr int kRollPitch = 20;                 // floats per strip row: the four rows of a step fall on different banks
constexpr int kRollFewRows = 64;               // up to this many rows the operand is gathered by the strips themselves
constexpr int kRollStripMax = 1792;            // rows a strip of 16 columns may have in LDS (140 KB)
template <int MAXM, bool DENSE>
__global__ __launch_bounds__(kRollStripThreads) void rollout_strip_kernel(const float* __restrict__ A,
                                                                          const float* __restrict__ G, int g_pitch,
                                                                          float* __restrict__ C,
                                                                          const int32_t* __restrict__ idx, int m, int L) {
  __shared__ float strip[MAXM * kRollPitch];
  __shared__ int32_t s_idx[DENSE ? 1 : MAXM];
  __shared__ unsigned in_s;                    // bit c: column c0 + c is in S
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  const int c0 = blockIdx.x * 16, col = c0 + r;
  const int mp = (m + 15) & ~15;
  if (tid == 0) in_s = 0u;
  __syncthreads();
  for (int i = tid; i < m; i += kRollStripThreads) {
    const int p = idx[i];
    if constexpr (!DENSE) s_idx[i] = p;
    if (p >= c0 && p < c0 + 16) atomicOr(&in_s, 1u << (p - c0));
  }
  for (int e = tid; e < mp * 16; e += kRollStripThreads) {
    const int i = e >> 4, c = e & 15;
    strip[i * kRollPitch + c] = i < m && c0 + c < L ? C[(size_t)i * L + c0 + c] : 0.f;
  }
  __syncthreads();
  for (int i0 = wave * 16; i0 < m; i0 += kRollStripWaves * 16) {
    const int arow = min(i0 + r, m - 1);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float direct[4];                             // requested in front of the contraction
#pragma unroll
    for (int j = 0; j < 4; ++j) direct[j] = A[(size_t)min(i0 + 4 * g + j, m - 1) * L + min(col, L - 1)];
    if constexpr (DENSE) {
      const float* grow = G + (size_t)arow * g_pitch + 4 * g;      // zero beyond column m
      f32x4 av[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) av[u] = *reinterpret_cast<const f32x4*>(grow + min(u * 16, mp - 16));
      for (int k0 = 0; k0 < mp; k0 += 64) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = k0 + u * 16;
          const f32x4 a = av[u];
          av[u] = *reinterpret_cast<const f32x4*>(grow + min(k + 64, mp - 16));
          if (k < mp) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], strip[(k + 4 * g + e) * kRollPitch + r], acc, 0, 0, 0);
          }
        }
      }
    } else {
      const float* a_row = A + (size_t)arow * L;
      float av[MAXM / 16][4];                    // the whole row's share of this lane, all loads in flight
#pragma unroll
      for (int u = 0; u < MAXM / 16; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) av[u][e] = a_row[s_idx[min(u * 16 + 4 * g + e, m - 1)]];
#pragma unroll
      for (int u = 0; u < MAXM / 16; ++u)
        if (u * 16 < mp) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int k = u * 16 + 4 * g + e;
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(k < m ? av[u][e] : 0.f, strip[k * kRollPitch + r], acc, 0, 0, 0);
          }
        }
    }
    if (col < L) {
      const bool own = in_s >> r & 1u;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = i0 + 4 * g + j;
        if (i >= m) break;
        C[(size_t)i * L + col] = 0.5f * (acc[j] + (own ? 0.f : direct[j]) + strip[i * kRollPitch + r]);
      }
    }
  }
}

// G[i, k] = A[i, S_k], pitch g_pitch = m rounded up to 16, zero beyond column m
__global__ __launch_bounds__(kRollThreads) void rollout_gather_kernel(const float* __restrict__ A,
                                                                      const int32_t* __restrict__ idx, int m, int L,
                                                                      int g_pitch, float* __restrict__ G) {
  const size_t e = (size_t)blockIdx.x * kRollThreads + threadIdx.x;
  if (e >= (size_t)m * g_pitch) return;
  const int i = (int)(e / g_pitch), k = (int)(e - (size_t)i * g_pitch);
  G[e] = k < m ? A[(size_t)i * L + idx[k]] : 0.f;
}

// More rows than a strip in LDS holds: not in place, one wave per 16 x 16 output tile (4 waves = 16 rows x 64 columns
// per workgroup), the operand gathered.
__global__ __launch_bounds__(kRollThreads) void rollout_kernel(const float* __restrict__ A,
                                                               const float* __restrict__ c_in,
                                                               float* __restrict__ c_out,
                                                               const int32_t* __restrict__ idx, int m, int L) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int i0 = blockIdx.y * 16;
  const int c0 = (blockIdx.x * 4 + wave) * 16;
  if (c0 >= L) return;
  const int arow = min(i0 + r, m - 1);
  const int bcol = min(c0 + r, L - 1);
  const float* a_row = A + (size_t)arow * L;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < m; k0 += 16) {
    float av[4], bv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = k0 + 4 * g + e;
      const bool ok = k < m;
      const int kk = ok ? k : m - 1;
      const float x = a_row[idx[kk]];
      av[e] = ok ? x : 0.f;
      bv[e] = c_in[(size_t)kk * L + bcol];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], bv[e], acc, 0, 0, 0);
  }
  const int col = c0 + r;
  if (col >= L) return;
  const bool in_s = find_sorted(idx, m, col) >= 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = i0 + 4 * g + j;
    if (i >= m) break;
    const float direct = in_s ? 0.f : A[(size_t)i * L + col];
    c_out[(size_t)i * L + col] = 0.5f * (acc[j] + direct + c_in[(size_t)i * L + col]);
  }
}

// Which of the 64 columns from c0 on lie in S, as a bitmap in LDS: every thread looks at its share of the index set (one
// memory latency instead of a search's ten).  All threads of the workgroup call it; ends on a barrier.
template <int THREADS>
__device__ __forceinline__ u64 columns_in_s(const int32_t* __restrict__ idx, int m, int c0, u64* word) {
  if (threadIdx.x == 0) *word = 0ull;
  __syncthreads();
  for (int i = threadIdx.x; i < m; i += THREADS) {
    const int p = idx[i];
    if (p >= c0 && p < c0 + 64) atomicOr(word, 1ull << (p - c0));
  }
  __syncthreads();
  return *word;
}

// Eq. 9 on the compact block: c_j = [j not in S] + sum_i C_S[i, j].  64 columns per workgroup, its 16 waves split the
// rows (wave w: rows w, w + 16, ..), the waves' sums are added in wave order.  97 rows x 1823 columns: 24.6 us with a
// thread per column, 4.0 now.
constexpr int kInflThreads = 1024;
__global__ __launch_bounds__(kInflThreads) void influence_kernel(const float* __restrict__ c_block,
                                                                 const int32_t* __restrict__ idx, int m, int L,
                                                                 float* __restrict__ influence) {
  __shared__ float red[kInflThreads / 64][64];
  __shared__ u64 word;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c0 = blockIdx.x * 64, col = c0 + lane;
  constexpr int NW = kInflThreads / 64;
  const float* ccol = c_block + min(col, L - 1);
  float s = 0.f;
  int i = wave;
  for (; i + 7 * NW < m; i += 8 * NW) {
    float x[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = ccol[(size_t)(i + t * NW) * L];
#pragma unroll
    for (int t = 0; t < 8; ++t) s += x[t];
  }
  for (; i < m; i += NW) s += ccol[(size_t)i * L];
  red[wave][lane] = s;
  const u64 own = columns_in_s<kInflThreads>(idx, m, c0, &word);
  if (wave != 0 || col >= L) return;
  s = own >> lane & 1ull ? 0.f : 1.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) s += red[w][lane];
  influence[col] = s;
}

// ------------------------------------------------------------------ Eq. 9 without the rollout matrix
// c = 1^T C^(N) = 1^T W^(N) W^(N-1) ... W^(1) (Eq. 8-9): multiplying from the LEFT keeps a length-L row
// vector v instead of the |S| x L block, O(m L) work per layer instead of O(m^2 L), at the price of needing
// the layers in reverse order, i.e. every layer's A-bar kept until the last one is done.  With rows outside
// S of W equal to unit vectors and rows i in S equal to (A-bar_i + e_i)/2 (Eq. 6-7):
//   (v W)_j = ( sum_{i in S} v_i A-bar_ij + ([j not in S] + 1) v_j ) / 2.
// Only the m entries u = v[S] feed back into later products; a column j outside S just accumulates:
//   u^(N) = ones;  u^(l-1)_k = ( sum_i u^(l)_i A-bar^(l)[i, S_k] + u^(l)_k ) / 2      (sequential, m x m per layer)
//   c_j = 1 + sum_l sum_i u^(l)_i A-bar^(l)[i, j] / 2   for j outside S,   c_{S_k} = u^(0)_k  (parallel)
// so the sequential part touches m^2 numbers per layer and the m L part is one fully parallel launch.
constexpr int kChainThreads = 1024;
constexpr int kChainMaxLen = 4096;           // = the selection kernel's length limit
constexpr int kChainFewRows = 128;           // up to this many rows a wave's share of a layer's block fits its registers
constexpr int kChainFewVals = 16;            // = kChainFewRows / (1024 / 128) rows per wave at most
constexpr int kChainSpreadMinRows = 129;     // from this many rows on the sequential part runs as a launch per layer

// The sequences one chain covers (independent: own A-bar slots, index set and influence vector); their dense
// blocks and per-layer vectors sit one after the other in the scratch buffers.
constexpr int kChainMaxSeqs = 8;
struct ChainSeq {
  const float* abar;
  const int32_t* idx;
  float* influence;
  int m, L;
  size_t g_off, u_off;          // in floats: n_layers * (sum of m^2, resp. of m, over the sequences before)
};
struct ChainSeqs {
  ChainSeq seq[kChainMaxSeqs];
};

// G[l][i, k] = abar[l][i, S_k]: the m x m blocks the sequential part reads, made dense first (all layers in
// one launch) so that the one workgroup that walks the layers reads consecutive floats.
__global__ __launch_bounds__(256) void chain_gather_kernel(const ChainSeqs seqs, size_t layer_stride,
                                                           float* __restrict__ g_scratch) {
  const ChainSeq& q = seqs.seq[blockIdx.z];
  const int m = q.m, L = q.L;
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t mm = (size_t)m * m;
  if (e >= mm) return;
  const int i = (int)(e / m), k = (int)(e - (size_t)i * m);
  g_scratch[q.g_off + (size_t)blockIdx.y * mm + e] = q.abar[(size_t)blockIdx.y * layer_stride + (size_t)i * L + q.idx[k]];
}

// Sequential part, one workgroup per sequence: u through the layers in reverse order; writes U[l][i] = u^(l)_i (the
// vector entering layer l) for the parallel part and c at the positions of S.  Items of 64 entries of S x
// one of RG row groups keep all 16 waves busy for short S; fixed summation order.
__global__ __launch_bounds__(kChainThreads) void chain_rows_kernel(const ChainSeqs seqs, int n_layers,
                                                                   const float* __restrict__ g_scratch,
                                                                   float* __restrict__ u_scratch) {
  const ChainSeq& q = seqs.seq[blockIdx.x];
  const float* __restrict__ G = g_scratch + q.g_off;
  float* __restrict__ U = u_scratch + q.u_off;
  const int32_t* __restrict__ idx = q.idx;
  float* __restrict__ influence = q.influence;
  const int m = q.m;
  __shared__ float u[2][kChainMaxLen];
  __shared__ float part[kChainMaxLen];                 // [RG][padded m], RG * padded m <= max(padded m, 1024)
  __shared__ int32_t s_idx[kChainMaxLen];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  for (int i = tid; i < m; i += kChainThreads) {
    u[0][i] = 1.f;
    s_idx[i] = idx[i];
  }
  __syncthreads();
  const int n_cb = (m + 63) / 64, mp = n_cb * 64;
  const int RG = mp < kChainThreads ? kChainThreads / mp : 1;
  const int n_items = n_cb * RG;
  int cur = 0;
  if (m <= kChainFewRows) {
    // Few rows (the decode steps): every wave has at most one item of at most kChainFewVals rows, so its
    // values of the NEXT layer's block are requested before this layer's sums are exchanged: the chain then
    // runs at one LDS round trip per layer instead of a memory latency.  Same sums in the same order as below.
    const bool has_item = wave < n_items;
    const int cb = wave % n_cb, rg = wave / n_cb;
    const int k = cb * 64 + lane;
    const float* acol = G + min(k, m - 1);
    auto load_layer = [&](float (&x)[kChainFewVals], int l) {
      const float* a = acol + (size_t)l * m * m;
#pragma unroll
      for (int t = 0; t < kChainFewVals; ++t) x[t] = a[(size_t)min(rg + t * RG, m - 1) * m];
    };
    float xs[kChainFewVals], xn[kChainFewVals];
    load_layer(xs, n_layers - 1);
    for (int l = n_layers - 1; l >= 0; --l) {
      const float* uin = u[cur];
      float* uout = u[cur ^ 1];
      load_layer(xn, max(l - 1, 0));                       // unconditional: the last one re-reads layer 0
      for (int i = tid; i < m; i += kChainThreads) U[(size_t)l * m + i] = uin[i];
      if (has_item) {
        float acc = 0.f;
#pragma unroll
        for (int t = 0; t < kChainFewVals; ++t) {
          const int i = rg + t * RG;
          if (i < m) acc = fmaf(uin[i], xs[t], acc);
        }
        part[rg * mp + k] = acc;
      }
      __syncthreads();
      for (int kk = tid; kk < m; kk += kChainThreads) {
        float sum = 0.f;
        for (int g2 = 0; g2 < RG; ++g2) sum += part[g2 * mp + kk];
        uout[kk] = 0.5f * (sum + uin[kk]);
      }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < kChainFewVals; ++t) xs[t] = xn[t];
      cur ^= 1;
    }
    for (int kk = tid; kk < m; kk += kChainThreads) influence[s_idx[kk]] = u[cur][kk];
    return;
  }
  for (int l = n_layers - 1; l >= 0; --l) {
    const float* a = G + (size_t)l * m * m;
    const float* uin = u[cur];
    float* uout = u[cur ^ 1];
    for (int i = tid; i < m; i += kChainThreads) U[(size_t)l * m + i] = uin[i];
    for (int item = wave; item < n_items; item += kChainThreads / 64) {
      const int cb = item % n_cb, rg = item / n_cb;
      const int k = cb * 64 + lane;
      const float* acol = a + min(k, m - 1);
      float acc = 0.f;
      int i = rg;
      for (; i + 7 * RG < m; i += 8 * RG) {
        float x[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t] = acol[(size_t)(i + t * RG) * m];
#pragma unroll
        for (int t = 0; t < 8; ++t) acc = fmaf(uin[i + t * RG], x[t], acc);
      }
      for (; i < m; i += RG) acc = fmaf(uin[i], acol[(size_t)i * m], acc);
      part[rg * mp + k] = acc;
    }
    __syncthreads();
    for (int k = tid; k < m; k += kChainThreads) {
      float sum = 0.f;
      for (int rg = 0; rg < RG; ++rg) sum += part[rg * mp + k];
      uout[k] = 0.5f * (sum + uin[k]);
    }
    __syncthreads();
    cur ^= 1;
  }
  for (int k = tid; k < m; k += kChainThreads) influence[s_idx[k]] = u[cur][k];
}

// The sequential part for long index sets (step 0, select-all): one launch per layer, 64 entries of S per
// workgroup, so that a layer's m x m product is spread over m / 64 compute units instead of one.  The vector
// entering layer l is U[l] (ones for the last layer, written here); the result goes to U[l - 1], or, after
// layer 0, to c at the positions of S.  A lane owns one entry k, the 16 waves split the rows i (wave w: rows
// w, w + 16, ..), the waves' sums are added in wave order: fixed summation order.
__global__ __launch_bounds__(kChainThreads) void chain_layer_kernel(const ChainSeqs seqs, int n_layers, int l,
                                                                    const float* __restrict__ g_scratch,
                                                                    float* __restrict__ u_scratch) {
  const ChainSeq& q = seqs.seq[blockIdx.y];
  const int m = q.m;
  if ((int)blockIdx.x * 64 >= m) return;                  // the grid follows the longest index set
  __shared__ float red[kChainThreads / 64][64];
  const float* __restrict__ G = g_scratch + q.g_off + (size_t)l * m * m;
  float* __restrict__ U = u_scratch + q.u_off;
  const float* __restrict__ uin = U + (size_t)l * m;
  const bool first = l == n_layers - 1;                   // u = ones
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int k = blockIdx.x * 64 + lane;
  const float* acol = G + min(k, m - 1);
  constexpr int NW = kChainThreads / 64;
  float acc = 0.f;
  int i = wave;
  for (; i + 7 * NW < m; i += 8 * NW) {
    float x[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = acol[(size_t)(i + t * NW) * m];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc = fmaf(first ? 1.f : uin[i + t * NW], x[t], acc);
  }
  for (; i < m; i += NW) acc = fmaf(first ? 1.f : uin[i], acol[(size_t)i * m], acc);
  red[wave][lane] = acc;
  __syncthreads();
  if (wave != 0 || k >= m) return;
  float sum = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) sum += red[w][lane];
  const float uk = first ? 1.f : uin[k];
  const float out = 0.5f * (sum + uk);
  if (first) U[(size_t)l * m + k] = 1.f;
  if (l > 0) U[(size_t)(l - 1) * m + k] = out;
  else q.influence[q.idx[k]] = out;
}

// Parallel part: 64 columns per workgroup, its 16 waves take the layers round-robin (wave w: layers w,
// w + 16, ..), a lane owns one column and adds u^(l)_i A-bar^(l)[i, j] over the rows in order with eight
// loads in flight; the waves' sums are added in wave order.  Columns inside S are left alone.
__global__ __launch_bounds__(kChainThreads) void chain_cols_kernel(const ChainSeqs seqs, size_t layer_stride,
                                                                   int n_layers,
                                                                   const float* __restrict__ u_scratch) {
  const ChainSeq& q = seqs.seq[blockIdx.y];
  const float* __restrict__ abar = q.abar;
  const int32_t* __restrict__ idx = q.idx;
  const float* __restrict__ U = u_scratch + q.u_off;
  float* __restrict__ influence = q.influence;
  const int m = q.m, L = q.L;
  if ((int)blockIdx.x * 64 >= L) return;                  // the grid follows the longest sequence
  __shared__ float red[kChainThreads / 64][64];
  __shared__ u64 word;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int col = blockIdx.x * 64 + lane;
  // nothing to do where every column is in S (a first step: all of them; 24 us for 512 rows before)
  const u64 outside = ~columns_in_s<kChainThreads>(idx, m, blockIdx.x * 64, &word) & low_mask(L - (int)blockIdx.x * 64);
  if (outside == 0ull) return;
  const float* acol = abar + min(col, L - 1);
  float acc = 0.f;
  for (int l = wave; l < n_layers; l += kChainThreads / 64) {
    const float* a = acol + (size_t)l * layer_stride;
    const float* ul = U + (size_t)l * m;
    int i = 0;
    for (; i + 16 <= m; i += 16) {                          // sixteen rows' loads in flight
      float x[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) x[t] = a[(size_t)(i + t) * L];
#pragma unroll
      for (int t = 0; t < 16; ++t) acc = fmaf(ul[i + t], x[t], acc);
    }
    for (; i < m; ++i) acc = fmaf(ul[i], a[(size_t)i * L], acc);
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave != 0 || !(outside >> lane & 1ull)) return;
  float sum = 0.f;
#pragma unroll
  for (int w = 0; w < kChainThreads / 64; ++w) sum += red[w][lane];
  influence[col] = 1.f + 0.5f * sum;
}

__global__ void ones_kernel(float* __restrict__ x, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = 1.f;
}

// ------------------------------------------------------------------ two-stage selection, one workgroup
constexpr int kSelThreads = 1024;            // seq_reset_kernel
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelMaxL = 4096;
constexpr int kSelT = 512;                    // threads of select_kernel: 8 waves (16 were slower: every wave scans for itself)
constexpr int kSelNW = kSelT / 64;
constexpr int kRankMax = 256;                // up to this many stage-1 candidates are ranked by counting
constexpr int kMergeMaxRows = 256;           // up to this many logit rows select_kernel merges Eq. 1's chunks (200 rows
                                             // cost it about 4 us, a launch for them 7.5; past 32 rows a wave it grows on)
constexpr int kMergeLaunchRows = 64;         // more rows: a launch of their own, so many rows a workgroup
static_assert(kMergeMaxRows / kSelNW <= 32 && kMergeLaunchRows <= kMergeMaxRows, "merge_rows holds 32 rows a wave");

struct SelShared {
  int wcnt[kSelWaves];
};

// Ordered compaction of {i in [0,n) : pred(i)} into out (ascending); returns the count (uniform).
template <typename Pred, typename Emit>
__device__ int block_compact(int n, Pred pred, Emit emit, SelShared* sh) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int base = 0;
  for (int start = 0; start < n; start += kSelThreads) {
    const int i = start + tid;
    const bool f = i < n && pred(i);
    const unsigned long long ballot = __ballot(f);
    const int before = __popcll(ballot & ((1ull << lane) - 1ull));
    __syncthreads();
    if (lane == 0) sh->wcnt[wave] = __popcll(ballot);
    __syncthreads();
    int off = 0, total = 0;
    for (int w = 0; w < kSelWaves; ++w) {
      const int c = sh->wcnt[w];
      if (w < wave) off += c;
      total += c;
    }
    if (f) emit(base + off + before, i);
    base += total;
  }
  __syncthreads();
  return base;
}

__device__ __forceinline__ u64 make_key(uint32_t bits, int index) {
  return ((u64)bits << 32) | (u64)(0xFFFFFFFFu - (unsigned)index);
}
__device__ __forceinline__ u64 bits_mass(uint32_t bits) {
  // floor(c * 2^32): the scaling is exact in float, the conversion truncates a non-negative value
  return (u64)(__uint_as_float(bits) * 4294967296.0f);
}
// Running totals over the wave with lane moves inside the vector ALU (no LDS round trip): lane i gets
// op(x_0, .., x_i), `zero` being op's neutral value.  HALVES: the two halves of the wave apart.
template <bool HALVES = false, typename Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, uint32_t zero, Op op) {
#define D2C_DPP(ctrl, rows) x = op(x, (uint32_t)__builtin_amdgcn_update_dpp((int)zero, (int)x, ctrl, rows, 0xf, false))
  D2C_DPP(0x111, 0xf);                     // from 1, 2, 4, 8 lanes below, inside rows of 16
  D2C_DPP(0x112, 0xf);
  D2C_DPP(0x114, 0xf);
  D2C_DPP(0x118, 0xf);
  D2C_DPP(0x142, 0xa);                     // last lane of rows 0, 2 into rows 1, 3
  if constexpr (!HALVES) D2C_DPP(0x143, 0xc);                     // lane 31 into rows 2, 3
#undef D2C_DPP
  return x;
}
__device__ __forceinline__ u64 wave_scan_add(u64 x) {
#define D2C_DPP(ctrl, rows)                                                                                      \
  x += (u64)(uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, ctrl, rows, 0xf, false) |                 \
       (u64)(uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), ctrl, rows, 0xf, false) << 32
  D2C_DPP(0x111, 0xf);
  D2C_DPP(0x112, 0xf);
  D2C_DPP(0x114, 0xf);
  D2C_DPP(0x118, 0xf);
  D2C_DPP(0x142, 0xa);
  D2C_DPP(0x143, 0xc);
#undef D2C_DPP
  return x;
}
// Value of one lane (the same lane for the whole wave) in every lane.
__device__ __forceinline__ uint32_t lane_of(uint32_t x, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)x, lane); }
__device__ __forceinline__ u64 lane_of(u64 x, int lane) {
  return (u64)lane_of((uint32_t)x, lane) | (u64)lane_of((uint32_t)(x >> 32), lane) << 32;
}
// Exclusive sum over the lanes below, of one value per lane; *total is the sum over the wave.
__device__ __forceinline__ uint32_t wave_before(uint32_t v, uint32_t* total) {
  const uint32_t incl = wave_scan(v, 0u, [](uint32_t p, uint32_t q) { return p + q; });
  *total = lane_of(incl, 63);
  return incl - v;
}

struct SelRadix {
  u64 hist[3][256];          // hist[*buf] is all zero between calls
  u64 sum[kSelNW];           // per wave: weights, OR and AND of the keys
  uint32_t any[kSelNW], all[kSelNW];
};

// Block-wide sum of w and OR / AND of kb over the live elements (one barrier; uniform results).
template <int PER>
__device__ void sel_reduce(const uint32_t (&kb)[PER], unsigned live, const u64 (&w)[PER], SelRadix& sh, u64* sum_out,
                           uint32_t* any_out, uint32_t* all_out) {
  u64 s = 0ull;
  uint32_t any = 0u, all = 0xffffffffu;
#pragma unroll
  for (int e = 0; e < PER; ++e)
    if (live >> e & 1u) {
      s += w[e];
      any |= kb[e];
      all &= kb[e];
    }
  s = wave_scan_add(s);
  any = wave_scan(any, 0u, [](uint32_t p, uint32_t q) { return p | q; });
  all = wave_scan(all, 0xffffffffu, [](uint32_t p, uint32_t q) { return p & q; });
  if ((threadIdx.x & 63) == 63) {
    sh.sum[threadIdx.x >> 6] = s;
    sh.any[threadIdx.x >> 6] = any;
    sh.all[threadIdx.x >> 6] = all;
  }
  __syncthreads();
  s = 0ull;
  any = 0u;
  all = 0xffffffffu;
#pragma unroll
  for (int v = 0; v < kSelNW; ++v) {
    s += sh.sum[v];
    any |= sh.any[v];
    all &= sh.all[v];
  }
  *sum_out = s;
  *any_out = any;
  *all_out = all;
}

// Weighted selection without a sort: the largest key t with sum{w : kb >= t} > thr, and above = sum{w : kb > t}
// (so above <= thr).  Eight key bits per pass: the weights of the elements that match the bits found so far are
// added up per digit in LDS (integer sums: the order does not matter), then every wave scans the 256 sums from the
// top by itself, so a pass costs one barrier.  Leading bits that all keys share (any / all) are skipped.
// Needs sum{w} > thr.  The three histograms rotate: the next pass's one is cleared before this pass's barrier.
template <int PER>
__device__ void sel_radix(const uint32_t (&kb)[PER], unsigned live, const u64 (&w)[PER], uint32_t any, uint32_t all,
                          u64 thr, SelRadix& sh, int* buf_io, uint32_t* t_out, u64* above_out) {
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t diff = any ^ all;
  int rem = diff ? 32 - __clz((int)diff) : 0;
  uint32_t prefix = rem >= 32 ? 0u : (all >> rem) << rem;
  u64 above = 0ull;
  int buf = *buf_io;
  while (rem > 0) {
    const int width = min(8, rem), shift = rem - width;
    const int next = buf == 2 ? 0 : buf + 1;
    if (tid < 256) sh.hist[next][tid] = 0ull;
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if ((live >> e & 1u) && (rem >= 32 || ((kb[e] ^ prefix) >> rem) == 0u))
        atomicAdd(&sh.hist[buf][(kb[e] >> shift) & ((1u << width) - 1u)], w[e]);
    __syncthreads();
    u64 h[4], s = 0ull;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h[i] = sh.hist[buf][255 - 4 * lane - i];
      s += h[i];
    }
    u64 run = above + wave_scan_add(s) - s;
    int digit = -1;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (digit < 0) {
        if (run + h[i] > thr) digit = 255 - 4 * lane - i;
        else run += h[i];
      }
    // the first lane that crosses; its run holds the weight above the digit
    const u64 cross = __ballot(digit >= 0);
    const int src = cross ? __builtin_ctzll(cross) : 0;
    prefix |= (lane_of((uint32_t)digit, src) & 0xffu) << shift;
    above = lane_of(run, src);
    rem = shift;
    buf = next;
  }
  *buf_io = buf;
  *t_out = prefix;
  *above_out = above;
}

constexpr int kKnownPad = 66;                // words: longest sequence and one window of 32 positions

constexpr int kSelMaxBatch = 8;
struct SelectBatch {
  SelectArgs seq[kSelMaxBatch];
};

// Eq. 1's chunks of a row -> confidence and prediction, by 32 lanes (64 with more than 32 chunks), two rows of a wave at a
// time; kSelT threads, at most kMergeMaxRows rows.  A row's sum is a scan over its lanes: the same bits for any number of rows.
// conf_s, pred_s (optional): the same by position in LDS.
__device__ void merge_rows(const SelectArgs& a, int wave, float* conf_s, int* pred_s) {
  const int lane = threadIdx.x & 63;
  const int width = a.n_chunks <= 32 ? 32 : 64, per = 64 / width;
  const int li = lane & (width - 1), sub = width == 32 ? lane >> 5 : 0;
  // lane q: position of the wave's q-th row (at most kMergeMaxRows / kSelNW = 32 rows a wave), one latency for all
  int where = 0;
  {
    const int row = (wave + (lane / per) * kSelNW) * per + lane % per;
    if (row < a.n_rows) where = a.via ? a.via[a.pos[row]] : a.pos[row];
  }
  constexpr int U = 4;                                       // rows of a wave whose triples are requested together
  float nm[U], np[U];
  int ni[U];
  auto fetch = [&](int row0) {                               // past the end: the last triple, not used
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int row = min(row0 + u * kSelNW * per + sub, a.n_rows - 1);
      const float* p = a.part + ((size_t)row * a.n_chunks + min(li, a.n_chunks - 1)) * 3;
      nm[u] = p[0];
      ni[u] = __float_as_int(p[1]);
      np[u] = p[2];
    }
  };
  // a reduction over the 32 (64) lanes of a row ends in the row's last lane; every lane reads it back from there
  auto spread = [&](uint32_t x) {
    const uint32_t lo = lane_of(x, 31), hi = lane_of(x, 63);
    return width == 32 && lane < 32 ? lo : hi;
  };
  auto reduce = [&](uint32_t x, uint32_t zero, auto op) {
    return spread(width == 32 ? wave_scan<true>(x, zero, op) : wave_scan<false>(x, zero, op));
  };
  fetch(wave * per);
  for (int row0 = wave * per, q = 0; row0 < a.n_rows; row0 += U * kSelNW * per) {
    float cm[U], cp[U];
    int ci[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { cm[u] = nm[u]; cp[u] = np[u]; ci[u] = ni[u]; }
    fetch(row0 + U * kSelNW * per);                          // fly during these rows' merges
#pragma unroll
    for (int u = 0; u < U; ++u, q += per) {
      const int row = row0 + u * kSelNW * per + sub;
      const bool on = row < a.n_rows && li < a.n_chunks;
      const float mine = on ? cm[u] : -INFINITY;
      const float best = __uint_as_float(reduce(__float_as_uint(mine), 0xff800000u, [](uint32_t x, uint32_t y) {
        return __float_as_uint(fmaxf(__uint_as_float(x), __uint_as_float(y)));
      }));
      const uint32_t bidx = reduce(on && mine == best ? (uint32_t)ci[u] : 0x7fffffffu, 0x7fffffffu,
                                   [](uint32_t x, uint32_t y) { return min(x, y); });
      const float sum = __uint_as_float(reduce(__float_as_uint(on ? cp[u] * expf(mine - best) : 0.f), 0u, [](uint32_t x, uint32_t y) {
        return __float_as_uint(__uint_as_float(x) + __uint_as_float(y));
      }));
      const int to = __shfl(where, (q + sub) & 63, kWave);
      if (on && li == 0) {
        const float conf = 1.0f / sum;
        a.conf[to] = conf;
        a.pred[to] = (int)bidx;
        if (conf_s) {
          conf_s[to] = conf;
          pred_s[to] = (int)bidx;
        }
      }
    }
  }
}

__global__ __launch_bounds__(kSelT) void confidence_merge_kernel(SelectArgs a) {
  const int row0 = blockIdx.x * kMergeLaunchRows;
  a.part += (size_t)row0 * a.n_chunks * 3;
  a.pos += row0;
  a.n_rows = min(kMergeLaunchRows, a.n_rows - row0);
  merge_rows(a, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nullptr, nullptr);
}

// One workgroup per sequence; the sequences are independent.  Latency is what bounds the selection (a few KB of
// input), so it is built from few barriers: the sets live as bitmaps of 64-position words in LDS (wave w of the
// workgroup ballots word e * waves + w for its e-th position), every wave turns a bitmap into counts and compaction
// offsets by itself (lane = word), and both selections look for a threshold key by radix (sel_radix) instead of sorting.
// Eq. 3's sum stops where the Gaussian is exactly zero in float.  Measured against a bitonic sort, rank counting, a
// scan per set and 16 waves (Eq. 1's merge then took another 5 / 7.5 us launch): L 512, 16 logit rows, 32 candidates
// 30.4 -> 14.8 us; L 3071, 200 logit rows, 737 candidates 327 -> 33 us.
// It has two halves.  The first (sel_first: Eq. 3's sums, and stage 2 where its candidates are the known tokens) needs no
// logits: it runs beside Eq. 1's chunks as workgroups of their launch and leaves its result in a SelPre.  The second (sel_second)
// merges the chunks, ranks, and emits the sets.  Chunks and selection one after the other, against halves: L 512, 16 logit rows of
// 126464 5.0 + 13.5 us -> 7.9 (the first half is the longer one) + 6.4; L 3071, 200 rows of 152064 22.6 + 32.5 -> 25.3 + 20.0.
// A call without logit rows, with cand_mode 1 or in a group of more sequences than a launch takes runs both in one kernel, with the
// block found once and the confidences read where they are needed (L 3071 without rows 30.5 us a call; as two halves behind each other 31.9).
// PER positions a thread: 1, 2, 4 or 8 for up to 512, 1024, 2048, 4096 positions.
struct SelPre {                                // what the first half leaves for the second
  u64 mask[64], u[64];                         // masked positions, stage-2 set: bitmaps
  float density[kSelMaxL];                     // Eq. 3, per candidate in ascending order
};

// The current block and its masked tokens (every wave for itself; lane = word of the bitmap); their positions go into cand.
struct SelBlock {
  int lo, hi, n_masked, n;
};
template <int PER>
__device__ __forceinline__ SelBlock sel_block(const SelectArgs& a, u64 mask_w, uint16_t* cand, int wave) {
  constexpr int T = kSelT, NW = kSelNW;
  const int tid = threadIdx.x, lane = tid & 63, L = a.L;
  const u64 below = low_mask(lane);
  SelBlock s;
  uint32_t n_masked_u;
  (void)wave_before((uint32_t)__popcll(mask_w), &n_masked_u);
  s.n_masked = (int)n_masked_u;
  s.lo = s.hi = L;
  if (s.n_masked > 0) {
    const int fw = __builtin_ctzll(__ballot(mask_w != 0ull));
    const int first_masked = fw * 64 + __builtin_ctzll(lane_of(mask_w, fw));
    // blocks are counted from the end of the prompt in both directions (floor division): a masked
    // position inside the prompt -- nothing the decoding loop produces, but a legal input -- lies in a
    // block with a negative number, cut at position 0
    const int diff = first_masked - a.prompt_len;
    const int b = diff >= 0 ? diff / a.block_len : -((-diff + a.block_len - 1) / a.block_len);
    const int64_t lo_raw = (int64_t)a.prompt_len + (int64_t)b * a.block_len;
    s.lo = (int)max((int64_t)0, lo_raw);
    s.hi = (int)min((int64_t)L, lo_raw + a.block_len);
  }
  const u64 cand_w = mask_w & low_mask(s.hi - lane * 64) & ~low_mask(s.lo - lane * 64);
  uint32_t n_u;
  const uint32_t before_w = wave_before((uint32_t)__popcll(cand_w), &n_u);
  s.n = (int)n_u;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int word = e * NW + wave;
    const u64 bits = lane_of(cand_w, word);
    const int before = (int)lane_of(before_w, word);
    if (bits >> lane & 1ull) cand[before + __popcll(bits & below)] = (uint16_t)(e * T + tid);
  }
  return s;
}

// Phases 3, 4: the smallest set of stage-2 candidates (the positions outside the bitmap `out`), by descending influence
// (lowest index first among equals), whose mass exceeds floor(p * total).  Leaves the set in w_u; ends on a barrier.
template <int PER>
__device__ __forceinline__ void sel_stage2(const SelectArgs& a, const float (&inf)[PER], u64 out_w, SelRadix& radix, int* buf, u64* w_tie,
                                           u64* w_u, int wave) {
  constexpr int T = kSelT, NW = kSelNW;
  const int tid = threadIdx.x, lane = tid & 63, L = a.L;
  const u64 below = low_mask(lane);
  uint32_t kb[PER];
  u64 mass[PER];
  unsigned live = 0u;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const u64 out = lane_of(out_w, e * NW + wave);
    kb[e] = __float_as_uint(inf[e]);
    mass[e] = 0ull;
    if (e * T + tid < L && !(out >> lane & 1ull)) {
      live |= 1u << e;
      mass[e] = bits_mass(kb[e]);
    }
  }
  unsigned in_u = live;
  if (a.p < 1.0f) {
    u64 total, above;
    uint32_t any, all, t;
    sel_reduce(kb, live, mass, radix, &total, &any, &all);
    const u64 thr = (u64)floor((double)a.p * __ull2double_rn(total));
    if (total > thr) {
      sel_radix(kb, live, mass, any, all, thr, radix, buf, &t, &above);
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const u64 word = __ballot((live >> e & 1u) && kb[e] == t);
        if (lane == 0) w_tie[e * NW + wave] = word;
      }
      __syncthreads();
      const u64 tie_w = lane < PER * NW ? w_tie[lane] : 0ull;
      uint32_t n_tie;
      const uint32_t tie_before = wave_before((uint32_t)__popcll(tie_w), &n_tie);
      u64 ties = 1ull;                                         // how many of the equal keys; a division only for a run
      if (n_tie > 1u) ties = (thr - above) / max(bits_mass(t), (u64)1) + 1ull;
      in_u = 0u;
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const int word = e * NW + wave;
        const u64 bits = lane_of(tie_w, word);
        const u64 rank = (u64)(lane_of(tie_before, word) + (uint32_t)__popcll(bits & below));
        if ((live >> e & 1u) && (kb[e] > t || (kb[e] == t && rank < ties))) in_u |= 1u << e;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const u64 word = __ballot(in_u >> e & 1u);
    if (lane == 0) w_u[e * NW + wave] = word;
  }
  __syncthreads();
}

template <int PER>
struct SelFirstLds {
  // room for shares of the sums; not less than for 2048 positions, so that a candidate's sum has one order up to there
  static constexpr int kDensity = PER * kSelT < 2048 ? 2048 : PER * kSelT;
  alignas(16) float phi[PER * kSelT + 32];
  float density[kDensity];
  u64 known[3 * kKnownPad];                    // known positions, with kKnownPad empty words on either side
  u64 mask[64], tie[64], u[64];
  uint16_t cand[PER * kSelT];
  SelRadix radix;
};

// What a thread has of the first half.  In a whole selection conf is requested behind Eq. 1's merge and used behind Eq. 3.
template <int PER>
struct SelOwn {
  float density[PER];                          // Eq. 3 of candidates t, t + T, ..
  float inf[PER];                              // influence at positions t, t + T, ..
  float conf[PER];                             // confidence of candidates t, t + T, ..
};

// The half without logits.  Leaves the candidates and the bitmaps mask and, with cand_mode 0, u in sh, behind a barrier.  WHOLE: the
// other half follows in this kernel; Eq. 1's chunks are merged here, the scores cleared.  buf: the radix buffer to go on with.
template <int PER, bool WHOLE>
__device__ __forceinline__ SelBlock sel_first(const SelectArgs& a, SelFirstLds<PER>& sh, SelOwn<PER>& mine, int& buf, int wave) {
  constexpr int T = kSelT, NW = kSelNW, ML = SelFirstLds<PER>::kDensity;
  const int L = a.L, tid = threadIdx.x, lane = tid & 63;
  // ---- mask flags and the Gaussian of Eq. 3.  score_out may be the influence's buffer: that is read first
  for (int i = tid; i < 256; i += T) sh.radix.hist[0][i] = 0ull;
  for (int i = tid; i < 3 * kKnownPad; i += T)
    if (i < kKnownPad || i >= kKnownPad + PER * NW) sh.known[i] = 0ull;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = e * T + tid;
    const bool f = j < L && a.is_masked[j] != 0;
    mine.inf[e] = j < L ? a.influence[j] : 0.f;
    const u64 word = __ballot(f), known = __ballot(j < L && !f);
    if (lane == 0) {
      sh.mask[e * NW + wave] = word;
      sh.known[kKnownPad + e * NW + wave] = known;
    }
    if (WHOLE && j < L && a.score_out) a.score_out[j] = 0.f;
  }
  for (int i = PER * NW + tid; i < 64; i += T) sh.mask[i] = sh.u[i] = 0ull;
  const float inv2s2 = 1.0f / (2.0f * a.sigma * a.sigma);
  // exp(-x) is zero in float from x = 104 on, subnormals included: distances of cut and more add nothing
  const int cut = (int)fminf((float)L, ceilf(sqrtf(105.0f / inv2s2)) + 1.0f);
  const int n_win = (cut + 31) >> 5;
  for (int d = tid; d < n_win * 32; d += T) sh.phi[d] = d < cut ? expf(-((float)d * (float)d) * inv2s2) : 0.f;
  if (WHOLE && a.part) merge_rows(a, wave, nullptr, nullptr);
  __syncthreads();
  const u64 mask_w = sh.mask[lane];
  const SelBlock blk = sel_block<PER>(a, mask_w, sh.cand, wave);
  const int n1 = blk.n;
  __syncthreads();
  if constexpr (WHOLE) {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int i = e * T + tid;
      mine.conf[e] = i < n1 ? a.conf[sh.cand[i]] : 0.f;
    }
  }

  // ---- phase 1: Eq. 3 on the masked tokens of the current block.  A wave takes 64 candidates (one a lane) and a share of
  // the distances, 32 at a time: the known positions at those distances are two 32-bit windows of the bitmap, phi is the
  // same for every lane, and a term costs three instructions.  Far distances are added first (the terms grow), left and
  // right, even and odd apart.
  const int n1p = (n1 + 63) & ~63;
  const int shares = n1 > 0 ? max(1, min(min(8, n_win), ML / n1p)) : 1;
  for (int item = wave; item < (n1p >> 6) * shares; item += NW) {
    const int q = item % shares, c = (item / shares) * 64 + lane;
    const int i = sh.cand[min(c, n1 - 1)];
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
    for (int w = q + ((n_win - 1 - q) / shares) * shares; w >= 0; w -= shares) {
      const int d0 = w * 32;
      auto window = [&](int p) {                               // known flags of positions p .. p + 31
        const unsigned at_bit = (unsigned)(p + kKnownPad * 64);
        const u64 lo_w = sh.known[at_bit >> 6], hi_w = sh.known[(at_bit >> 6) + 1];
        const unsigned s = at_bit & 63u;
        return (uint32_t)(lo_w >> s) | (s ? (uint32_t)(hi_w << (64u - s)) : 0u);
      };
      const uint32_t right = window(i + d0), left = window(i - d0 - 31);
#pragma unroll
      for (int b = 31; b >= 0; --b) {
        const uint32_t f = __float_as_uint(sh.phi[d0 + b]);
        sum[(b & 1) * 2] += __uint_as_float(f & (uint32_t)((int32_t)(right << (31 - b)) >> 31));
        sum[(b & 1) * 2 + 1] += __uint_as_float(f & (uint32_t)((int32_t)(left << b) >> 31));
      }
    }
    sh.density[q * n1p + c] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
  }
  if (a.cand_mode == 0) sel_stage2<PER>(a, mine.inf, mask_w, sh.radix, &buf, sh.tie, sh.u, wave);
  else __syncthreads();
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int c = e * T + tid;
    mine.density[e] = 0.f;
    if (c < n1)
      for (int q = shares - 1; q >= 0; --q) mine.density[e] += sh.density[q * n1p + c];
  }
  return blk;
}

struct SelSecondLds {
  u64 tie[64], mst[64], dec[64], u[64];
  u64 rkey[kRankMax], dkey[kRankMax];
  int n_small;
};
// and with the first half's result from memory: what else that half has
template <int PER>
struct SelSplitLds {
  float conf[PER * kSelT];
  int pred[PER * kSelT];
  uint16_t cand[PER * kSelT];
  SelRadix radix;
};

// The half behind Eq. 1, and all of it with SPLIT false (own: SelFirstLds then, SelSplitLds otherwise).
template <int PER, bool SPLIT, typename Own>
__device__ __forceinline__ void sel_second(const SelectArgs& a, SelSecondLds& sh, Own& own, int wave) {
  constexpr int T = kSelT, NW = kSelNW;
  const int L = a.L, tid = threadIdx.x, lane = tid & 63;
  const u64 below = low_mask(lane);
  int buf = 0;
  u64 mask_w, u_w = 0ull;
  SelOwn<PER> mine;
  SelBlock blk;
  for (int i = tid; i < 64; i += T) sh.mst[i] = sh.dec[i] = sh.u[i] = sh.tie[i] = 0ull;
  if constexpr (SPLIT) {
    const SelPre* pre = static_cast<const SelPre*>(a.pre);
    mask_w = pre->mask[lane];
    u_w = pre->u[lane];
#pragma unroll
    for (int e = 0; e < PER; ++e) mine.density[e] = pre->density[e * T + tid];      // of candidate e T + tid, if there are so many
    for (int i = tid; i < 256; i += T) own.radix.hist[0][i] = 0ull;
    // confidences and predictions so far, then Eq. 1's chunks of this call's logit rows over them
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int j = e * T + tid;
      if (j < L) {
        own.conf[j] = a.conf[j];
        own.pred[j] = a.pred[j];
        if (a.score_out) a.score_out[j] = 0.f;
      }
    }
    __syncthreads();
    if (a.part) merge_rows(a, wave, own.conf, own.pred);
    blk = sel_block<PER>(a, mask_w, own.cand, wave);
    __syncthreads();
  } else {
    blk = sel_first<PER, true>(a, own, mine, buf, wave);
    mask_w = own.mask[lane];
    if (a.cand_mode == 0) u_w = own.u[lane];
  }
  const int n1 = blk.n;

  // ---- phase 2: Eq. 4 (top-k) and the decode set on D(i) * s^i; thread t holds candidates t, t + T, ..  The decode set ranks
  // the same scores, or the confidences alone (conf_decode), and with a threshold also takes every candidate whose confidence
  // exceeds it.
  int at[PER];
  float cf[PER];
  unsigned clive = 0u;
  uint32_t sb[PER], db[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int c = e * T + tid;
    at[e] = 0;
    cf[e] = 0.f;
    sb[e] = db[e] = 0u;
    if (c < n1) {
      clive |= 1u << e;
      at[e] = own.cand[c];
      if constexpr (SPLIT) cf[e] = own.conf[at[e]];
      else cf[e] = mine.conf[e];
      const float score = mine.density[e] * cf[e];
      sb[e] = __float_as_uint(score);
      db[e] = a.conf_decode ? __float_as_uint(cf[e]) : sb[e];
      if (a.score_out) a.score_out[at[e]] = score;
    }
  }
  unsigned in_m = a.k >= n1 ? clive : 0u, in_d = a.n_unmask >= n1 ? clive : 0u;
  const bool cut_m = a.k > 0 && a.k < n1, cut_d = a.n_unmask > 0 && a.n_unmask < n1;
  if (n1 <= kRankMax) {
    if (cut_m || cut_d) {                                    // rank by counting (n1 <= T: at most one candidate a thread)
      if (tid < n1) {
        sh.rkey[tid] = make_key(sb[0], at[0]);
        sh.dkey[tid] = make_key(db[0], at[0]);
      }
      __syncthreads();
      if (tid < n1) {
        const u64 mine = sh.rkey[tid], dmine = sh.dkey[tid];
        int rank = 0, drank = 0;
        for (int o = 0; o < n1; ++o) {
          rank += sh.rkey[o] > mine ? 1 : 0;
          drank += sh.dkey[o] > dmine ? 1 : 0;
        }
        if (cut_m && rank < a.k) in_m |= 1u;
        if (cut_d && drank < a.n_unmask) in_d |= 1u;
      }
    }
  } else {
    // the count-th largest key by radix; candidates with an equal key are taken in ascending order
    auto top = [&](const uint32_t (&kb)[PER], int count) {
      u64 ones[PER], sum, above;
      uint32_t any, all, t;
#pragma unroll
      for (int e = 0; e < PER; ++e) ones[e] = 1ull;
      sel_reduce(kb, clive, ones, own.radix, &sum, &any, &all);
      sel_radix(kb, clive, ones, any, all, (u64)(count - 1), own.radix, &buf, &t, &above);
      const int ties = count - (int)above;                   // >= 1
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const u64 word = __ballot((clive >> e & 1u) && kb[e] == t);
        if (lane == 0) sh.tie[e * NW + wave] = word;
      }
      __syncthreads();
      const u64 tie_w = sh.tie[lane];
      uint32_t n_tie;
      const uint32_t tie_before = wave_before((uint32_t)__popcll(tie_w), &n_tie);
      unsigned f = 0u;
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const int word = e * NW + wave;
        const u64 bits = lane_of(tie_w, word);
        const int rank = (int)lane_of(tie_before, word) + __popcll(bits & below);
        if ((clive >> e & 1u) && (kb[e] > t || (kb[e] == t && rank < ties))) f |= 1u << e;
      }
      __syncthreads();                                       // tie and the reduction slots are used again
      return f;
    };
    if (cut_m) in_m = top(sb, a.k);
    if (cut_d && !a.conf_decode && cut_m && a.n_unmask <= a.k && a.k <= kRankMax) {
      // the same ranking, and the decode set lies inside M*: count ranks among those k
      if (tid == 0) sh.n_small = 0;
      __syncthreads();
#pragma unroll
      for (int e = 0; e < PER; ++e)
        if (in_m >> e & 1u) sh.rkey[atomicAdd(&sh.n_small, 1)] = make_key(sb[e], at[e]);      // exactly k of them, in any order
      __syncthreads();
#pragma unroll
      for (int e = 0; e < PER; ++e)
        if (in_m >> e & 1u) {
          const u64 mine = make_key(sb[e], at[e]);
          int rank = 0;
          for (int o = 0; o < a.k; ++o) rank += sh.rkey[o] > mine ? 1 : 0;
          if (rank < a.n_unmask) in_d |= 1u << e;
        }
    } else if (cut_d) {
      in_d = top(db, a.n_unmask);
    }
  }
#pragma unroll
  for (int e = 0; e < PER; ++e)
    if (clive >> e & 1u) {
      const u64 bit = 1ull << (at[e] & 63);
      if (in_m >> e & 1u) atomicOr(&sh.mst[at[e] >> 6], bit);
      if ((in_d >> e & 1u) || (a.threshold > 0.f && cf[e] > a.threshold)) atomicOr(&sh.dec[at[e] >> 6], bit);
    }
  __syncthreads();
  const u64 mst_w = sh.mst[lane], dec_w = sh.dec[lane];
  if (!SPLIT && a.cand_mode != 0) {                          // stage 2's candidates: everything outside M*
    sel_stage2<PER>(a, mine.inf, mst_w, own.radix, &buf, sh.tie, sh.u, wave);
    u_w = sh.u[lane];
  }

  // ---- phase 5: unmask (Eq. 2), emit M*, I_t, U, S_{t+1} = M* u I_t u U and its still-masked rows: all offsets from
  // the bitmaps (two counts of at most 4096 to a register)
  const u64 s_w = mst_w | dec_w | u_w, row_w = s_w & mask_w & ~dec_w;
  uint32_t tot_a, tot_b, tot_c;
  const uint32_t pre_a = wave_before((uint32_t)__popcll(mst_w) | (uint32_t)__popcll(dec_w) << 16, &tot_a);
  const uint32_t pre_b = wave_before((uint32_t)__popcll(u_w) | (uint32_t)__popcll(s_w) << 16, &tot_b);
  const uint32_t pre_c = wave_before((uint32_t)__popcll(row_w), &tot_c);
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = e * T + tid, word = e * NW + wave;
    const u64 m_b = lane_of(mst_w, word), d_b = lane_of(dec_w, word), u_b = lane_of(u_w, word);
    const u64 s_b = lane_of(s_w, word), r_b = lane_of(row_w, word);
    const uint32_t pa = lane_of(pre_a, word), pb = lane_of(pre_b, word), pc = lane_of(pre_c, word);
    if (m_b >> lane & 1ull) a.mstar[(pa & 0xffffu) + __popcll(m_b & below)] = j;
    if (d_b >> lane & 1ull) {
      a.decode_idx[(pa >> 16) + __popcll(d_b & below)] = j;
      if constexpr (SPLIT) a.tokens[j] = own.pred[j];
      else a.tokens[j] = a.pred[j];
      a.is_masked[j] = 0;
    }
    if (u_b >> lane & 1ull) a.u_set[(pb & 0xffffu) + __popcll(u_b & below)] = j;
    if (s_b >> lane & 1ull) {
      const int slot = (int)(pb >> 16) + __popcll(s_b & below);
      a.s_next[slot] = j;
      if (r_b >> lane & 1ull) a.s_rows_next[pc + __popcll(r_b & below)] = slot;
    }
  }
  if (tid == 0) {
    a.counts[0] = (int)(tot_a & 0xffffu);
    a.counts[1] = (int)(tot_b & 0xffffu);
    a.counts[2] = (int)(tot_b >> 16);
    a.counts[3] = (int)(tot_a >> 16);
    a.counts[4] = (int)tot_c;
    a.counts[5] = blk.n_masked - (int)(tot_a >> 16);
    a.counts[6] = blk.lo;
    a.counts[7] = blk.hi;
  }
}

template <int PER, bool SPLIT>
__global__ __launch_bounds__(kSelT) void select_kernel(const SelectBatch batch) {
  __shared__ SelSecondLds sh;
  __shared__ std::conditional_t<SPLIT, SelSplitLds<PER>, SelFirstLds<PER>> own;
  sel_second<PER, SPLIT>(batch.seq[blockIdx.x], sh, own, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

// Eq. 1's chunks alone, one a workgroup: where the launch has no first half beside them (pieces of a group but the last, cand_mode 1,
// a second stream, many sequences).  Memory bounds it; the barriers of two chunks and the registers of a first half cost 4 us on 256
// rows of 126464 (the Eq. 1 and selection launches of 1200 masked rows 159 us in the kernel below, 144 in this one).
template <bool VEC>
__global__ __launch_bounds__(kConfThreads) void confidence_chunk_kernel(const float* __restrict__ logits, int vocab, int chunk, int n_chunks,
                                                                        float* __restrict__ part) {
  __shared__ ConfLds lds;
  if constexpr (VEC) confidence_chunk_vec(logits, vocab, n_chunks, part, blockIdx.y, blockIdx.x, lds);
  else confidence_chunk(logits, vocab, chunk, n_chunks, part, blockIdx.y, blockIdx.x, lds);
}

// Eq. 1's chunks, and in front of them the halves without logits of n_first selections: one workgroup each, which runs as long
// as the chunks of a few dozen rows or longer, so it goes first.  A workgroup has the selection's 8 waves; four make a chunk.
// Six waves a SIMD: with 117 registers, four, the loads in flight did not fill the memory's queue (200 rows 28.5 us, 25.3 now).
template <int PER, bool VEC>
__global__ __launch_bounds__(kSelT, 6) void confidence_select_kernel(const float* __restrict__ logits, int vocab, int chunk, int n_chunks,
                                                                  int n_rows, float* __restrict__ part, const SelectBatch batch,
                                                                  int n_first) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if ((int)blockIdx.x < n_first) {
    __shared__ SelFirstLds<PER> sh;
    const SelectArgs& a = batch.seq[blockIdx.x];
    SelPre* pre = static_cast<SelPre*>(a.pre);
    SelOwn<PER> mine;
    int buf = 0;
    (void)sel_first<PER, false>(a, sh, mine, buf, wave);
    const int tid = threadIdx.x;
    if (tid < 64) {
      pre->mask[tid] = sh.mask[tid];
      pre->u[tid] = sh.u[tid];
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) pre->density[e * kSelT + tid] = mine.density[e];      // those behind the last are not used
    return;
  }
  __shared__ ConfLds lds[kSelT / kConfThreads];
  const int half = wave / (kConfThreads / 64), item = ((int)blockIdx.x - n_first) * 2 + half;
  const int at = min(item, n_rows * n_chunks - 1);           // an odd count: the last chunk twice, the same numbers
  const int row = at / n_chunks, ck = at - row * n_chunks;
  if constexpr (VEC) confidence_chunk_vec(logits, vocab, n_chunks, part, row, ck, lds[half]);
  else confidence_chunk(logits, vocab, chunk, n_chunks, part, row, ck, lds[half]);
}

// Step-0 state: S_0 = all rows, s_rows = masked rows, conf = 0, pred = 0.
__global__ __launch_bounds__(kSelThreads) void seq_reset_kernel(const uint8_t* __restrict__ is_masked, int L,
                                                                int32_t* __restrict__ s_idx,
                                                                int32_t* __restrict__ s_rows,
                                                                float* __restrict__ conf, int32_t* __restrict__ pred,
                                                                int32_t* __restrict__ counts) {
  __shared__ SelShared sh;
  for (int j = threadIdx.x; j < L; j += kSelThreads) {
    s_idx[j] = j;
    conf[j] = 0.f;
    pred[j] = 0;
  }
  const int n = block_compact(L, [&](int j) { return is_masked[j] != 0; },
                              [&](int slot, int j) { s_rows[slot] = j; }, &sh);
  if (threadIdx.x == 0) {
    for (int c = 0; c < 8; ++c) counts[c] = 0;
    counts[2] = L;
    counts[4] = n;
    counts[5] = n;
  }
}

}  // namespace

int select_max_len() { return kSelMaxL; }


int confidence_chunks(int vocab) {
  int chunk = kConfChunk;
  while ((vocab + chunk - 1) / chunk > kConfMaxChunks) chunk *= 2;
  return (vocab + chunk - 1) / chunk;
}

size_t confidence_scratch_floats(size_t n_rows, int vocab) { return n_rows * confidence_chunks(vocab) * 3; }

static_assert(sizeof(SelPre) == kSelPreFloats * sizeof(float), "what callers keep for a first half");

// positions a thread of the selection for sequences of up to max_L positions
static int sel_per(int max_L) { return max_L <= kSelT ? 1 : max_L <= 2 * kSelT ? 2 : max_L <= 4 * kSelT ? 4 : 8; }

hipError_t launch_confidence_chunks(const float* logits, int n_rows, int vocab, float* part, hipStream_t st, const SelectArgs* first,
                                    int n_first) {
  if (n_rows <= 0) return n_first > 0 ? hipErrorInvalidValue : hipSuccess;
  if (vocab <= 0 || part == nullptr || n_first < 0 || n_first > kSelMaxBatch) return hipErrorInvalidValue;
  int chunk = kConfChunk;
  while ((vocab + chunk - 1) / chunk > kConfMaxChunks) chunk *= 2;
  const int n_chunks = confidence_chunks(vocab);
  const bool vec = chunk == kConfChunk && vocab % 4 == 0 && vocab >= 4 && (uintptr_t)logits % 16 == 0;
  if (n_first == 0) {
    const dim3 grid(n_chunks, n_rows), threads(kConfThreads);
    if (vec) hipLaunchKernelGGL(confidence_chunk_kernel<true>, grid, threads, 0, st, logits, vocab, chunk, n_chunks, part);
    else hipLaunchKernelGGL(confidence_chunk_kernel<false>, grid, threads, 0, st, logits, vocab, chunk, n_chunks, part);
    return hipGetLastError();
  }
  SelectBatch batch;
  int max_L = 1;
  for (int i = 0; i < n_first; ++i) {
    if (first[i].L <= 0 || first[i].L > kSelMaxL || first[i].block_len <= 0 || first[i].prompt_len < 0 ||
        first[i].prompt_len > first[i].L || first[i].cand_mode != 0 || !first[i].pre)
      return hipErrorInvalidValue;
    batch.seq[i] = first[i];
    max_L = std::max(max_L, first[i].L);
  }
  for (int i = n_first; i < kSelMaxBatch; ++i) batch.seq[i] = SelectArgs{};
  const dim3 grid(n_first + (unsigned)(((size_t)n_rows * n_chunks + 1) / 2)), threads(kSelT);
#define D2C_CONF(PER_)                                                                                                         \
  do {                                                                                                                         \
    if (vec)                                                                                                                   \
      hipLaunchKernelGGL((confidence_select_kernel<PER_, true>), grid, threads, 0, st, logits, vocab, chunk, n_chunks, n_rows, \
                         part, batch, n_first);                                                                                \
    else                                                                                                                       \
      hipLaunchKernelGGL((confidence_select_kernel<PER_, false>), grid, threads, 0, st, logits, vocab, chunk, n_chunks,        \
                         n_rows, part, batch, n_first);                                                                        \
    return hipGetLastError();                                                                                                  \
  } while (0)
  switch (sel_per(max_L)) {
    case 1: D2C_CONF(1);
    case 2: D2C_CONF(2);
    case 4: D2C_CONF(4);
    default: D2C_CONF(8);
  }
#undef D2C_CONF
}

bool rollout_in_place(int layer, int m) { return layer == 0 || m <= kRollStripMax; }
size_t rollout_scratch_floats(int max_m) { return (size_t)max_m * ((max_m + 15) & ~15); }

hipError_t launch_rollout(const float* attn_avg, float* c_block, float* scratch, const int32_t* idx, int m, int L,
                          bool first, hipStream_t st) {
  if (m <= 0) return hipSuccess;
  if (first) {
    hipLaunchKernelGGL(rollout_first_kernel, dim3((L + kRollThreads - 1) / kRollThreads, m), dim3(kRollThreads), 0, st,
                       attn_avg, c_block, idx, m, L);
    return hipGetLastError();
  }
  const dim3 strips((L + 15) / 16), threads(kRollStripThreads);
  if (m <= kRollFewRows) {
    hipLaunchKernelGGL((rollout_strip_kernel<kRollFewRows, false>), strips, threads, 0, st, attn_avg, nullptr, 0, c_block, idx, m, L);
    return hipGetLastError();
  }
  if (m <= kRollStripMax) {
    const int pitch = (m + 15) & ~15;
    hipLaunchKernelGGL(rollout_gather_kernel, dim3((unsigned)(((size_t)m * pitch + kRollThreads - 1) / kRollThreads)),
                       dim3(kRollThreads), 0, st, attn_avg, idx, m, L, pitch, scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (m <= 768)
      hipLaunchKernelGGL((rollout_strip_kernel<768, true>), strips, threads, 0, st, attn_avg, scratch, pitch, c_block, idx, m, L);
    else
      hipLaunchKernelGGL((rollout_strip_kernel<kRollStripMax, true>), strips, threads, 0, st, attn_avg, scratch, pitch, c_block, idx, m, L);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(rollout_kernel, dim3((L + 63) / 64, (m + 15) / 16), dim3(kRollThreads), 0, st, attn_avg, c_block,
                     scratch, idx, m, L);
  return hipGetLastError();
}

hipError_t launch_influence(const float* c_block, const int32_t* idx, int m, int L, float* influence,
                            hipStream_t st) {
  if (L <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(influence_kernel, dim3((L + 63) / 64), dim3(kInflThreads), 0, st, c_block, idx, m, L, influence);
  return hipGetLastError();
}

int chain_max_batch() { return kChainMaxSeqs; }

hipError_t launch_influence_chain(const ChainCall* calls, int n_calls, size_t layer_stride, int n_layers,
                                  float* u_scratch, float* g_scratch, hipStream_t st) {
  if (n_calls <= 0) return hipSuccess;
  if (n_calls > kChainMaxSeqs || n_layers < 0) return hipErrorInvalidValue;
  ChainSeqs seqs;
  std::memset(&seqs, 0, sizeof(seqs));
  int n = 0, max_m = 0, max_L = 0;
  size_t g_off = 0, u_off = 0;
  for (int i = 0; i < n_calls; ++i) {
    const ChainCall& c = calls[i];
    if (c.L <= 0 || c.L > kChainMaxLen || c.m < 0 || c.m > c.L) return hipErrorInvalidValue;
    if (c.m == 0 || n_layers == 0) {         // nothing was refreshed: C = I, every c_j = 1
      hipLaunchKernelGGL(ones_kernel, dim3((c.L + 255) / 256), dim3(256), 0, st, c.influence, c.L);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      continue;
    }
    seqs.seq[n++] = ChainSeq{c.abar, c.idx, c.influence, c.m, c.L, g_off, u_off};
    g_off += (size_t)n_layers * c.m * c.m;
    u_off += (size_t)n_layers * c.m;
    max_m = std::max(max_m, c.m);
    max_L = std::max(max_L, c.L);
  }
  if (n == 0) return hipSuccess;
  const size_t mm = (size_t)max_m * max_m;
  hipLaunchKernelGGL(chain_gather_kernel, dim3((unsigned)((mm + 255) / 256), n_layers, n), dim3(256), 0, st, seqs,
                     layer_stride, g_scratch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (max_m >= kChainSpreadMinRows) {
    // long index sets: a launch per layer over m / 64 workgroups beats one workgroup walking all layers
    for (int l = n_layers - 1; l >= 0; --l) {
      hipLaunchKernelGGL(chain_layer_kernel, dim3((max_m + 63) / 64, n), dim3(kChainThreads), 0, st, seqs, n_layers, l,
                         g_scratch, u_scratch);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  } else {
    hipLaunchKernelGGL(chain_rows_kernel, dim3(n), dim3(kChainThreads), 0, st, seqs, n_layers, g_scratch, u_scratch);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(chain_cols_kernel, dim3((max_L + 63) / 64, n), dim3(kChainThreads), 0, st, seqs, layer_stride,
                     n_layers, u_scratch);
  return hipGetLastError();
}

int select_max_batch() { return kSelMaxBatch; }

hipError_t launch_select(const SelectArgs* args, int n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (n > kSelMaxBatch) return hipErrorInvalidValue;
  SelectBatch batch;
  int max_L = 0;
  for (int i = 0; i < n; ++i) {
    const SelectArgs& a = args[i];
    if (a.L <= 0 || a.L > kSelMaxL || a.block_len <= 0 || a.prompt_len < 0 || a.prompt_len > a.L)
      return hipErrorInvalidValue;
    if (a.n_rows < 0 || (a.n_rows > 0 && (!a.part || !a.pos || a.n_chunks <= 0 || a.n_chunks > kConfMaxChunks)))
      return hipErrorInvalidValue;
    if ((a.pre != nullptr) != (args[0].pre != nullptr) || (a.pre && a.cand_mode != 0)) return hipErrorInvalidValue;
    batch.seq[i] = a;
    if (a.n_rows == 0) batch.seq[i].part = nullptr;
    if (a.n_rows > kMergeMaxRows) {
      // many logit rows: their chunks are merged by a launch of their own, spread over more than one compute unit
      hipLaunchKernelGGL(confidence_merge_kernel, dim3((a.n_rows + kMergeLaunchRows - 1) / kMergeLaunchRows), dim3(kSelT), 0, st, a);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      batch.seq[i].part = nullptr;
    }
    max_L = std::max(max_L, a.L);
  }
  for (int i = n; i < kSelMaxBatch; ++i) batch.seq[i] = args[0];        // never read: the grid has n workgroups
#define D2C_SELECT(PER_)                                                                                  \
  do {                                                                                                    \
    if (args[0].pre) hipLaunchKernelGGL((select_kernel<PER_, true>), dim3(n), dim3(kSelT), 0, st, batch); \
    else hipLaunchKernelGGL((select_kernel<PER_, false>), dim3(n), dim3(kSelT), 0, st, batch);            \
    return hipGetLastError();                                                                             \
  } while (0)
  switch (sel_per(max_L)) {
    case 1: D2C_SELECT(1);
    case 2: D2C_SELECT(2);
    case 4: D2C_SELECT(4);
    default: D2C_SELECT(8);
  }
#undef D2C_SELECT
}

hipError_t launch_seq_reset(const uint8_t* is_masked, int L, int32_t* s_idx, int32_t* s_rows, float* conf,
                            int32_t* pred, int32_t* counts, hipStream_t st) {
  if (L <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(seq_reset_kernel, dim3(1), dim3(kSelThreads), 0, st, is_masked, L, s_idx, s_rows, conf, pred,
                     counts);
  return hipGetLastError();
}

}  // namespace d2c
