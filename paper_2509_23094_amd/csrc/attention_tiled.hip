// Selective-refresh attention for MANY query rows (a long selected set, step 0, the
// isolated attention op with m = 256): the regime where the m x L x d_h contraction
// is at the matrix-core / HBM ridge rather than bound by streaming K and V once.
// Same mathematics as the few-row kernels (Sec. 4.2 of the d2Cache paper: the selected
// queries attend to all L cached keys without a mask, and A-bar is the head mean of the
// normalised rows), different blocking:
//
//   forward   one workgroup = 64*QT (or 128*QT) query rows of one head over one range of keys.
//             K and V blocks of 64 keys are staged through LDS once per workgroup, in whole rows, the next
//             block's on their way during the arithmetic; V is transposed as it is read from there.
//             Scores are computed transposed (S^T = K Q^T) so the accumulator of two 16-key tiles IS the
//             32-key B operand of O^T += V^T P^T.  Both contractions use the 16x16x32 step.
//             When the grid would not fill the chip the key range is split; every split writes
//             an unnormalised fp32 partial with its running maximum and sum, and a merge
//             kernel combines them in a fixed order (bit-reproducible, no atomics).
//   A-bar     from the probabilities that the forward kernel leaves behind (EMIT), in the launch that also merges the splits.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "common.h"
#include "internal.h"

namespace d2c {
namespace {

constexpr int kThreads = 256;
constexpr int kBlockKeys = 64;
// rows of the unnormalised probabilities are padded by one block: the pitch between heads and rows is then no
// power of two (the head average reads the same piece of every head at once)
constexpr int kPtildePad = 64;

// two floats -> one register of two bf16 (round to nearest even): a single packed conversion
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// One sequence of a batched launch (blockIdx.y picks it): its tensors, sizes, launch plan and scratch pieces.
struct SeqArgs {
  const bf16 *q, *k_cache, *v_cache;
  bf16* out;
  float *lse, *attn_avg, *o_part, *ml_part, *refblk;
  bf16* ptilde;
  int m, L, keys_per_split, n_splits, q_blocks, avg_blocks;
};
constexpr int kMaxBatch = 8;             // sequences per launch (the arguments travel by value)
struct BatchArgs {
  SeqArgs seq[kMaxBatch];
};

// Workgroup id -> (query block, head, key split).  Ids are dealt round-robin to the 8 XCDs; the query
// blocks that share one (head, split), i.e. the same K and V bytes, get consecutive slots of ONE XCD.
struct TileId {
  int qb, head, split;
  bool valid;
};
__device__ __forceinline__ TileId tile_of(int bid, int q_blocks, int n_heads, int n_splits) {
  const int xcd = bid & 7, slot = bid >> 3;
  const int tile = (slot / q_blocks) * 8 + xcd;
  TileId t;
  t.qb = slot % q_blocks;
  t.head = tile / n_splits;
  t.split = tile - t.head * n_splits;
  t.valid = tile < n_heads * n_splits;
  return t;
}

// EMIT: the kernel also writes what the head average needs, so that no second pass over Q and K is run:
// the unnormalised probabilities of every block exactly as they enter the matrix cores (bf16,
// ptilde [H, m, Lp], Lp = L rounded up to whole blocks; inside a block of 64 keys the values of a row sit in
// operand order: 16-byte piece (ks, g) holds keys 32ks + 4g .. +3, then 32ks + 16 + 4g .. +3) and the base-2
// reference each block was taken against (refblk [H, blocks, m]).  The head-average kernel turns them into normalised rows once the rows'
// log-sum-exp is known: p = ptilde * 2^(refblk - lse2).
//
// WAVES = 4 or 8 waves per workgroup, each owning 16*QT queries.  Two waves share a SIMD, so that one wave's
// matrix-core phase runs beside the other's vector phase: two workgroups of 4 waves or one of 8 (two LDS buffers, 64 KB).
//
// K and V rows go from global memory straight into LDS (DMA), one block ahead, in whole rows; V is transposed on its way out of
// LDS (ds_read_b64_tr_b16).  Loads and stores retire in one queue, which is waited for once, in the middle of a
// block: the rows were requested at its start, the last block's probability stores behind the last wait.
// 1024 queries x 2048 keys, 32 heads, no average: 50 us, 0.69 PFLOP/s, in 256 workgroups of 4 waves.  Rows through registers
// took 94 us a layer for 4 x 228 x 3072 with the average (now 83), and for 777 x 777 without, unsplit, 31 (now 23; in the two splits
// it took then 51 with the merge): the compiler had moved their loads behind the scores and their wait in front of everything
// stored.  What is left: the probabilities (half of the time of a call with the average), the wait in mid-block (a row has half a block
// to arrive), and 1 to 2 waves per SIMD between whose phases a third of the time is idle.
// DMA = false brings the rows through registers: buffers that are not 16-byte aligned.
__device__ __forceinline__ u32x2 lds_read_transposed(const unsigned char* p) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
}

template <int DH, int QT, int WAVES, bool EMIT, bool DMA>
__global__ __launch_bounds__(WAVES * 64, 2) void attn_tiled_fwd_kernel(const BatchArgs batch, int n_heads, int n_kv_heads,
                                                                       float scale) {
  static_assert(WAVES == 4 || WAVES == 8, "4 or 8 waves");
  constexpr int NS = DH / 32;            // contraction steps of K Q^T
  constexpr int ND = DH / 16;            // head-dim tiles of O^T
  constexpr int kRow = DH * 2;                           // bytes of a K or V row
  constexpr int kOperand = kBlockKeys * kRow;            // bytes of a block's K (or V) rows
  constexpr int PP = kRow / 16;                          // 16-byte pieces of a row
  constexpr int RP = 64 / PP;                            // rows that one instruction of a wave brings
  constexpr int LP = kBlockKeys / RP / WAVES;            // instructions per wave and operand
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * 2 * kOperand];         // [buffer][K, V][key][piece]

  const SeqArgs& sq = batch.seq[blockIdx.y];
  const bf16* __restrict__ q = sq.q;
  bf16* __restrict__ out = sq.out;
  float* __restrict__ lse = sq.lse;
  float* __restrict__ o_part = sq.o_part;
  float* __restrict__ ml_part = sq.ml_part;
  const int m = sq.m, L = sq.L, keys_per_split = sq.keys_per_split, n_splits = sq.n_splits, q_blocks = sq.q_blocks;
  const TileId id = tile_of(blockIdx.x, q_blocks, n_heads, n_splits);
  if (!id.valid || id.qb >= q_blocks) return;          // the grid is sized for the largest sequence of the batch
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  const int head = id.head;
  const int kvh = head / (n_heads / n_kv_heads);
  const int dq = n_heads * DH;
  const size_t kv_pitch = (size_t)n_kv_heads * DH;
  const int q0 = id.qb * (16 * QT * WAVES) + wave * (16 * QT);
  const bool active = q0 < m;                          // a wave without queries only stages
  const int key_lo = id.split * keys_per_split;
  const int key_hi = min(L, key_lo + keys_per_split);
  const int n_blocks = (key_hi - key_lo + kBlockKeys - 1) / kBlockKeys;      // >= 1 by the launch plan
  const int n_blk_total = (L + kBlockKeys - 1) / kBlockKeys;
  const int Lp = n_blk_total * kBlockKeys + kPtildePad;                      // row pitch of ptilde

  // Staging: PP neighbouring lanes bring one row.  In LDS the 16-byte pieces of a row are permuted by an xor with the row
  // number, so that the 16 rows of an operand read fall on different banks: single pieces of K, pairs of V (a transposed
  // read takes 32 bytes of a row).
  auto k_swz = [](int row) { return DH == 128 ? row & 15 : row >> 1 & 7; };
  auto v_swz = [](int row) { return (DH == 128 ? row & 7 : row >> 1 & 3) << 1; };
  const unsigned pitch = (unsigned)(kv_pitch * 2);
  const int srow = wave * RP + lane / PP, spc = lane % PP;      // first row and piece of this lane; further rows 16s on
  const int k_src = (spc ^ k_swz(srow)) * 16, v_src = (spc ^ v_swz(srow)) * 16;
  const bf16* kbase = sq.k_cache + (size_t)key_lo * kv_pitch + (size_t)kvh * DH;
  const bf16* vbase = sq.v_cache + (size_t)key_lo * kv_pitch + (size_t)kvh * DH;
  const int kv_bytes = (int)(unsigned)(((size_t)(key_hi - key_lo - 1) * kv_pitch + DH) * 2);
  const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(kbase), 0, kv_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(vbase), 0, kv_bytes, 0x00020000);
  u32x4 reg_k[LP], reg_v[LP];                                   // !DMA only
  auto load_block = [&](int blk, int buf) {
    const int key0 = blk * kBlockKeys, left = key_hi - key_lo - 1 - key0;       // rows past the end repeat the last one
    const bool whole = left >= kBlockKeys - 1;
    unsigned char* dst = lds + buf * (2 * kOperand) + wave * 1024;
#pragma unroll
    for (int j = 0; j < LP; ++j) {
      const int row = whole ? srow : min(srow + j * (RP * WAVES), left);
      const size_t first = (size_t)(key0 + (whole ? j * (RP * WAVES) : 0)) * pitch;
      if constexpr (DMA) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(krsrc, (__attribute__((address_space(3))) void*)(dst + j * (WAVES * 1024)), 16,
                                                 (int)(row * pitch + k_src), (int)(unsigned)first, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vrsrc, (__attribute__((address_space(3))) void*)(dst + kOperand + j * (WAVES * 1024)),
                                                 16, (int)(row * pitch + v_src), (int)(unsigned)first, 0, 0);
      } else {
        reg_k[j] = ld16(reinterpret_cast<const char*>(kbase) + first + (row * pitch + k_src));
        reg_v[j] = ld16(reinterpret_cast<const char*>(vbase) + first + (row * pitch + v_src));
      }
    }
  };
  auto store_block = [&](int buf) {                             // !DMA
    unsigned char* dst = lds + buf * (2 * kOperand) + wave * 1024 + lane * 16;
#pragma unroll
    for (int j = 0; j < LP; ++j) {
      *reinterpret_cast<u32x4*>(dst + j * (WAVES * 1024)) = reg_k[j];
      *reinterpret_cast<u32x4*>(dst + kOperand + j * (WAVES * 1024)) = reg_v[j];
    }
  };
  load_block(0, 0);

  // this wave's queries as B operands of S^T = K Q^T (rows past m repeat row m-1)
  Frag<bf16> qf[QT][NS];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int row = min(q0 + t * 16 + r, m - 1);
    const bf16* qrow = q + (size_t)row * dq + head * DH + g * 8;
#pragma unroll
    for (int s = 0; s < NS; ++s) qf[t][s].raw = ld16(qrow + s * 32);
  }

  // Where the probabilities go (rows past m store what row m-1 stores, to its place)
  const bool emits = EMIT && sq.ptilde != nullptr;              // null: a sequence of the batch whose average is not wanted
  char* prow[QT];
  char* rrow[QT];
  if constexpr (EMIT) {
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      const size_t row = (size_t)min(q0 + t * 16 + r, m - 1);
      const size_t blk0 = (size_t)(key_lo / kBlockKeys);        // key_lo is a multiple of the block length
      prow[t] = reinterpret_cast<char*>(sq.ptilde + ((size_t)head * m + row) * Lp + blk0 * kBlockKeys + 8 * g);
      rrow[t] = reinterpret_cast<char*>(sq.refblk + ((size_t)head * n_blk_total + blk0) * m + row);
    }
  }

  // Online softmax in the base-2 domain: p = 2^(s*c - ref) with c = scale*log2(e).  ref is a per-row
  // reference, not necessarily the running maximum: it is only raised (and O, l rescaled) when a score
  // exceeds it by more than kRaise, so p stays below 2^kRaise.  The result is the same softmax (shift
  // invariance).  Every lane checks its own 16 scores of a row against the row's reference; only when some lane
  // of the wave finds one too large do the four lanes that share a row exchange their maxima and raise the
  // reference (rare after the first block).  Both ask the same question in the same rounding, so that a row is
  // raised by its own scores, whichever rows share the wave.
  constexpr float kRaise = 8.f;
  const float c2 = scale * 1.44269504088896341f;
  float ref[QT], l_run[QT];
  f32x4 acc[ND][QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    ref[t] = -INFINITY;
    l_run[t] = 0.f;
#pragma unroll
    for (int d = 0; d < ND; ++d) acc[d][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  constexpr int kRing = 4;                     // LDS fragments in flight ahead of the matrix-core step that uses them
  // byte offsets of this lane's operand pieces (the step or head-dim tile enters by an xor, the key tile by an addition)
  const unsigned k_rd = r * kRow + (g ^ k_swz(r)) * 16;
  const int v_row = 4 * g + (r >> 2);
  const unsigned v_rd = kOperand + v_row * kRow + (v_swz(v_row) ^ (r >> 1 & 1)) * 16 + (r & 1) * 8;

  // everything this wave has requested from memory is there (vmcnt(0))
  auto wait_requests = [&]() {
    __builtin_amdgcn_s_waitcnt(0x70 | 0xf00);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto block = [&](int blk, int buf) {
    const unsigned char* kv = lds + buf * (2 * kOperand);
    const int key0 = key_lo + blk * kBlockKeys;
    f32x4 st[4][QT];
    // ---- scores S^T = K Q^T; the first step of every tile starts from a zero accumulator operand.
    // The K fragments come from LDS through a ring of kRing registers: fragment i + kRing is requested right
    // behind the matrix-core steps of fragment i, so one LDS latency is paid per block, not one per fragment
    // (the scheduler is told to keep this order; left alone it waits for every pair of reads).
    {
      constexpr int NF = 4 * NS;
      auto read_k = [&](int i) { return *reinterpret_cast<const u32x4*>(kv + (k_rd ^ (unsigned)(i % NS * 64)) + i / NS * (16 * kRow)); };
      Frag<bf16> kf[kRing];
#pragma unroll
      for (int i = 0; i < kRing; ++i) kf[i].raw = read_k(i);
#pragma unroll
      for (int i = 0; i < NF; ++i) {
#pragma unroll
        for (int t = 0; t < QT; ++t) {
          if (i % NS == 0)
            st[i / NS][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, kf[i % kRing].raw), __builtin_bit_cast(bf16x8, qf[t][0].raw),
                f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          else
            mfma16(st[i / NS][t], kf[i % kRing], qf[t][i % NS]);
        }
        if (i + kRing < NF) kf[i % kRing].raw = read_k(i + kRing);
      }
      __builtin_amdgcn_sched_group_barrier(0x100, kRing, 0);
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, QT, 0);
        if (i + kRing < NF) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    }
    if (key0 + kBlockKeys > key_hi) {    // ragged last block of the range: keys past the end score -inf
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (key0 + a * 16 + 4 * g + j >= key_hi) {
#pragma unroll
            for (int t = 0; t < QT; ++t) st[a][t][j] = -INFINITY;
          }
    }
    // ---- this lane's maxima against the rows' references
    float tmax[QT];
    bool need = false;
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      float am[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) am[a] = fmaxf(fmaxf(st[a][t][0], st[a][t][1]), fmaxf(st[a][t][2], st[a][t][3]));
      tmax[t] = fmaxf(fmaxf(am[0], am[1]), fmaxf(am[2], am[3]));
      need = need || tmax[t] * c2 > ref[t] + kRaise;
    }
    if (__builtin_amdgcn_ballot_w64(need) != 0) {
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        float rmax = fmaxf(tmax[t], __shfl_xor(tmax[t], 16, kWave));
        rmax = fmaxf(rmax, __shfl_xor(rmax, 32, kWave)) * c2;       // the row's maximum; -inf only if it has no key yet
        const float ref_new = rmax > ref[t] + kRaise ? rmax : ref[t];
        const float alpha = ref_new == ref[t] ? 1.f : __builtin_amdgcn_exp2f(ref[t] - ref_new);   // 0 on the first block
        l_run[t] *= alpha;
#pragma unroll
        for (int d = 0; d < ND; ++d) acc[d][t] *= alpha;
        ref[t] = ref_new;
      }
    }
    // ---- probabilities against the references, packed as the B operand of O^T += V^T P^T
    Frag<bf16> pf[2][QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      const float nref = -ref[t];
      float psum = 0.f;
      float x[4][4];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          x[a][j] = __builtin_amdgcn_exp2f(fmaf(st[a][t][j], c2, nref));
          psum += x[a][j];
        }
      l_run[t] += psum;                                // this lane's share; lanes are added at the end
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        pf[ks][t].raw = u32x4{pack_bf16(x[2 * ks][0], x[2 * ks][1]), pack_bf16(x[2 * ks][2], x[2 * ks][3]),
                              pack_bf16(x[2 * ks + 1][0], x[2 * ks + 1][1]),
                              pack_bf16(x[2 * ks + 1][2], x[2 * ks + 1][3])};
    }
    if constexpr (DMA) wait_requests();
    if constexpr (EMIT) {
      // a lane holds 4 consecutive keys of each of the block's 4 key tiles for query row r of tile t, stored as packed:
      // the 64 values of (row, block) in the order [32-key step][lane group][tile, key]
      if (emits) {
#pragma unroll
        for (int t = 0; t < QT; ++t) {
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
            *reinterpret_cast<u32x4*>(prow[t] + (size_t)blk * (kBlockKeys * 2) + ks * 64) = pf[ks][t].raw;
          *reinterpret_cast<float*>(rrow[t] + (size_t)blk * m * 4) = ref[t];       // the four lanes of a row store the same
        }
      }
    }
    // ---- O^T += V^T P^T, the V fragments through the same kind of ring
    {
      constexpr int NF = ND * 2;
      auto read_v = [&](int i) {           // head-dim tile i / 2, 32-key step i % 2: 4 keys of either 16-key tile
        const unsigned char* p = kv + (v_rd ^ (unsigned)(i / 2 * 32)) + i % 2 * (32 * kRow);
        const u32x2 lo = lds_read_transposed(p), hi = lds_read_transposed(p + 16 * kRow);
        return u32x4{lo.x, lo.y, hi.x, hi.y};
      };
      Frag<bf16> vf[kRing];
#pragma unroll
      for (int i = 0; i < kRing; ++i) vf[i].raw = read_v(i);
#pragma unroll
      for (int i = 0; i < NF; ++i) {
#pragma unroll
        for (int t = 0; t < QT; ++t) mfma16(acc[i / 2][t], vf[i % kRing], pf[i % 2][t]);
        if (i + kRing < NF) vf[i % kRing].raw = read_v(i + kRing);
      }
      __builtin_amdgcn_sched_group_barrier(0x100, 2 * kRing, 0);
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, QT, 0);
        if (i + kRing < NF) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
    }
  };

  auto barrier = [&]() {                       // without the wait for everything that __syncthreads() brings
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (DMA) {
    wait_requests();
    barrier();
  } else {
    store_block(0);
    __syncthreads();
  }
  for (int blk = 0; blk < n_blocks; ++blk) {
    const int buf = blk & 1;
    // the buffer that is filled now was last read one iteration ago, before the barrier every wave has passed
    if (blk + 1 < n_blocks) load_block(blk + 1, buf ^ 1);
    if constexpr (DMA) {
      __builtin_amdgcn_sched_barrier(0);
      if (active) block(blk, buf);
      else wait_requests();
      __builtin_amdgcn_sched_barrier(0);
      barrier();
    } else {
      if (active) block(blk, buf);
      if (blk + 1 < n_blocks) store_block(buf ^ 1);
      __syncthreads();
    }
  }
  if (!active) return;

#pragma unroll
  for (int t = 0; t < QT; ++t) {
    float l = l_run[t];
    l += __shfl_xor(l, 16, kWave);
    l += __shfl_xor(l, 32, kWave);
    const int row = q0 + t * 16 + r;
    if (row >= m) continue;
    const size_t prow = ((size_t)id.split * n_heads + head) * m + row;
    if (g == 0 && ml_part != nullptr && (EMIT || n_splits > 1)) {
      ml_part[prow * 2] = ref[t];                        // base-2 reference of this partial
      ml_part[prow * 2 + 1] = l;
    }
    if (n_splits == 1) {
      const float inv = 1.0f / l;
      bf16* dst = out + (size_t)row * dq + head * DH + 4 * g;
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        const u32x2 v = {pack_bf16(acc[d][t][0] * inv, acc[d][t][1] * inv),
                         pack_bf16(acc[d][t][2] * inv, acc[d][t][3] * inv)};
        *reinterpret_cast<u32x2*>(dst + d * 16) = v;
      }
      if (g == 0) lse[(size_t)head * m + row] = ref[t] * 0.693147180559945309f + __logf(l);
    } else {
      float* dst = o_part + prow * DH + 4 * g;
#pragma unroll
      for (int d = 0; d < ND; ++d) *reinterpret_cast<f32x4*>(dst + d * 16) = acc[d][t];
    }
  }
}

// Everything that has to wait for all key splits of a row, in one launch with two kinds of workgroups.
//   merge (the workgroups behind the first avg_blocks, only with several key splits):
//     out[row, head, :] = sum_s 2^{ref_s - M} O_s / sum_s 2^{ref_s - M} l_s in split order, and the row's log-sum-exp;
//   head average (the first avg_blocks workgroups): A-bar[i, j] = (1/H) sum_h ptilde[h, i, j] 2^{refblk[h, j / 64, i] - lse2[h, i]}, heads in
//     order, with lse2[h, i] = M + log2 sum_s l_s 2^{ref_s - M} (M = max_s ref_s) recomputed from the splits' (ref, l).
//     A workgroup takes kFinRows rows x kFinKeys keys; a thread owns 8 consecutive keys of one row.
constexpr int kFinRows = 2, kFinKeys = 1024, kFinHeads = 64;
template <int DH>
__global__ __launch_bounds__(kThreads) void attn_finish_kernel(const BatchArgs batch, int n_heads) {
  const SeqArgs& sq = batch.seq[blockIdx.y];
  const float* __restrict__ o_part = sq.o_part;
  const float* __restrict__ ml_part = sq.ml_part;
  const bf16* __restrict__ ptilde = sq.ptilde;
  const float* __restrict__ refblk = sq.refblk;
  bf16* __restrict__ out = sq.out;
  float* __restrict__ lse = sq.lse;
  float* __restrict__ attn_avg = sq.attn_avg;
  const int m = sq.m, L = sq.L, n_splits = sq.n_splits, avg_blocks = sq.avg_blocks;
  if ((int)blockIdx.x >= avg_blocks) {                    // the head-average workgroups run longest and go first
    if (n_splits <= 1) return;                            // nothing to merge (the grid is sized for the whole batch)
    constexpr int PER_ROW = DH / 4;                       // threads per (head, row): 4 values each
    const size_t item = (size_t)((int)blockIdx.x - avg_blocks) * kThreads + threadIdx.x;
    const size_t hr = item / PER_ROW;                     // head * m + row
    const int c = (int)(item - hr * PER_ROW);
    if (hr >= (size_t)n_heads * m) return;
    const int head = (int)(hr / m), row = (int)(hr - (size_t)head * m);
    float mx = -INFINITY;
    for (int s = 0; s < n_splits; ++s) mx = fmaxf(mx, ml_part[((size_t)s * n_heads * m + hr) * 2]);
    float lsum = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < n_splits; ++s) {
      const size_t prow = (size_t)s * n_heads * m + hr;
      const float f = __builtin_amdgcn_exp2f(ml_part[prow * 2] - mx);
      lsum += ml_part[prow * 2 + 1] * f;
      o += *reinterpret_cast<const f32x4*>(o_part + prow * DH + 4 * c) * f;
    }
    const float inv = 1.0f / lsum;
    const u32x2 v = {pack_bf16(o[0] * inv, o[1] * inv), pack_bf16(o[2] * inv, o[3] * inv)};
    *reinterpret_cast<u32x2*>(out + (size_t)row * n_heads * DH + head * DH + 4 * c) = v;
    if (c == 0) lse[hr] = mx * 0.693147180559945309f + __logf(lsum);
    return;
  }
  __shared__ float lse2_s[kFinHeads][kFinRows];
  const int n_blk = (L + kBlockKeys - 1) / kBlockKeys, Lk = n_blk * kBlockKeys, Lp = Lk + kPtildePad;
  const int key_tiles = (Lk + kFinKeys - 1) / kFinKeys;
  const int b = (int)blockIdx.x;
  const int rb = b / key_tiles, kb = b - rb * key_tiles;
  const int tid = threadIdx.x, rr = tid / (kFinKeys / 8), c = tid % (kFinKeys / 8);
  const int row = rb * kFinRows + rr;
  const int j0 = kb * kFinKeys + c * 8;                    // this thread's 16-byte piece of the row
  const bool live = row < m && j0 < Lk;
  const int rowc = min(row, m - 1), j0c = min(j0, Lk - 8);
  const bf16* pbase = ptilde + (size_t)rowc * Lp + j0c;
  const float* rbase = refblk + (size_t)(j0c >> 6) * m + rowc;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  constexpr int U = 32;                                    // heads per trip: their loads are issued together
  for (int h0 = 0; h0 < n_heads; h0 += kFinHeads) {
    const int nh = min(kFinHeads, n_heads - h0);
    // the first trip's loads are requested before the rows' log-sum-exp is put together, so that the two
    // latencies overlap (heads past the end repeat the last one and are not added)
    u32x4 pv[U];
    float rf[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t h = (size_t)(h0 + min(u, nh - 1));
      pv[u] = ld16(pbase + h * m * Lp);
      rf[u] = rbase[h * n_blk * m];
    }
    __syncthreads();
    for (int item = tid; item < kFinHeads * kFinRows; item += kThreads) {
      const int hh = item / kFinRows, r2 = item - hh * kFinRows;
      const int row2 = min(rb * kFinRows + r2, m - 1);
      if (hh < nh) {
        const size_t hr = (size_t)(h0 + hh) * m + row2;
        float ms[8], ls[8];                                  // at most 8 key splits
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const size_t prow = (size_t)min(s, n_splits - 1) * n_heads * m + hr;
          ms[s] = ml_part[prow * 2];
          ls[s] = ml_part[prow * 2 + 1];
        }
        float mx = ms[0];
#pragma unroll
        for (int s = 1; s < 8; ++s) mx = fmaxf(mx, ms[s]);
        float lsum = 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s)
          if (s < n_splits) lsum += ls[s] * __builtin_amdgcn_exp2f(ms[s] - mx);
        lse2_s[hh][r2] = mx + __builtin_amdgcn_logf(lsum);      // v_log_f32 is a base-2 logarithm
      }
    }
    __syncthreads();
    for (int hh = 0; hh < nh; hh += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (hh + u < nh) {
          const float f = __builtin_amdgcn_exp2f(rf[u] - lse2_s[hh + u][rr]);
          const bf16x8 pb = __builtin_bit_cast(bf16x8, pv[u]);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] = fmaf((float)pb[e], f, acc[e]);
        }
      }
      if (hh + U < nh) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const size_t h = (size_t)(h0 + min(hh + U + u, nh - 1));
          pv[u] = ld16(pbase + h * m * Lp);
          rf[u] = rbase[h * n_blk * m];
        }
      }
    }
  }
  if (!live) return;
  // piece (ks, g) of block blk holds keys 64 blk + 32 ks + 4 g .. +3 and the same 16 keys further on
  const float inv_h = 1.0f / (float)n_heads;
  const int piece = (j0 >> 3) & 7, ks = piece >> 2, g = piece & 3;
  const int key_a = (j0 & ~63) + 32 * ks + 4 * g, key_b = key_a + 16;
  float* dst = attn_avg + (size_t)row * L;
  if ((L & 3) == 0) {                                      // rows start 16-byte aligned
    if (key_a < L) *reinterpret_cast<f32x4*>(dst + key_a) = f32x4{acc[0] * inv_h, acc[1] * inv_h, acc[2] * inv_h, acc[3] * inv_h};
    if (key_b < L) *reinterpret_cast<f32x4*>(dst + key_b) = f32x4{acc[4] * inv_h, acc[5] * inv_h, acc[6] * inv_h, acc[7] * inv_h};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (key_a + e < L) dst[key_a + e] = acc[e] * inv_h;
      if (key_b + e < L) dst[key_b + e] = acc[4 + e] * inv_h;
    }
  }
}

// Tile shape and key splits of one launch.
struct FwdPlan {
  int qt, waves, splits;
  int q_per_wg() const { return 16 * qt * waves; }
};
// A sequence whose workgroups in the largest tile shape alone fill the chip is never split (the scratch is sized by this).
bool may_split(const Tunables& t, int m, int n_heads) { return ((m + 255) / 256) * n_heads < t.attn_target_wgs; }

// The cheapest by a model of the time in us.  A workgroup has a part per block of 64 keys, of the width of the heads: of 128, 1.8 for
// 4 waves alone on a compute unit, 2.8 where two workgroups share one, 2.6 for 8 waves (of twice the queries); of 64, 0.75 of that
// (1.30 / 1.73 measured alone, 0.96 / 1.40 without the head average).  Several splits write and read fp32 partials (about 3.5 TB/s
// both ways together), so a split pays only while compute units are idle: 777 rows x 777 keys, 32 heads of 128, 22 us unsplit, 36 in
// two; 256 x 2048 42 us, 26 in four, 33 in eight; heads of 64, 200 x 2048 18 us in four, 22 in eight by 8 waves.
// The parts are those of calls with the head average (1.35, 2.05 and 1.95 without, and the merge is then a launch of its own);
// the plan must not depend on it, since the output's bits may not.  Against the best of 1 to 8 splits by 4 and 8 waves, over 202 sizes of
// 16-1024 rows x 512-4096 keys, 16 to 32 heads: heads of 128 1.2 % above it on average (9 % of the sizes by more than 5, the worst
// 12 %), without the average 5 % (33 %, 51 %); heads of 64 0.8 % (4 %, 12 %) and 7 % (43 %, 55 %).
FwdPlan plan_fwd(const Tunables& t, const TiledCall* calls, int n_calls, int n_heads, int head_dim) {
  int max_m = 0, max_L = 0;
  double partial_us = 0.0;                        // of one split
  for (int i = 0; i < n_calls; ++i) {
    max_m = std::max(max_m, calls[i].m);
    max_L = std::max(max_L, calls[i].L);
    if (may_split(t, calls[i].m, n_heads)) partial_us += 8.0 * calls[i].m * n_heads * head_dim / 3.5e6;
  }
  const int qt = t.attn_qt == 1 || t.attn_qt == 2 ? t.attn_qt : (max_m > 64 ? 2 : 1);
  const int blocks = (std::max(1, max_L) + kBlockKeys - 1) / kBlockKeys;
  const int max_splits = std::min(std::max(1, std::min(8, t.attn_max_splits)), blocks);
  const int units = std::min(t.attn_target_wgs, 1 << 20);         // more than any launch has; twice this fits an int
  const double heads = head_dim == 64 ? 0.75 : 1.0, width = heads * (qt == 1 ? 0.55 : 1.0);      // 16 queries per wave
  const double alone = width * 1.8, shared = width * 2.8, eight = heads * 2.6;
  FwdPlan best{qt, t.attn_waves == 8 ? 8 : 4, 1};
  double best_us = 1e30;
  for (int waves : {4, 8}) {
    if ((waves == 8 && qt == 1) || (t.attn_waves != 0 && waves != t.attn_waves)) continue;
    for (int s = 1; s <= max_splits; ++s) {
      FwdPlan p{qt, waves, s};
      int wgs = 0;
      for (int i = 0; i < n_calls; ++i)
        wgs += (calls[i].m + p.q_per_wg() - 1) / p.q_per_wg() * n_heads * (may_split(t, calls[i].m, n_heads) ? s : 1);
      const int room = waves == 4 ? 2 * units : units;            // workgroups on the chip at one time
      const int rest = wgs % room;
      const double full = waves == 4 ? shared : eight;
      const double rounds = wgs / room * full + (rest == 0 ? 0.0 : waves == 4 && rest <= units ? alone : full);
      const double us = (blocks + s - 1) / s * rounds + (s > 1 ? s * partial_us : 0.0);
      if (us < best_us * 0.999) {
        best_us = us;
        best = p;
      }
    }
  }
  return best;
}

// Scratch of one call, in floats: partial outputs of the key splits, their (reference, sum) pairs, the
// unnormalised probabilities (bf16, two per float) and the per-block references.
struct Scratch {
  size_t o_part, ml, ptilde, refblk, total;
};
Scratch scratch_of(int n_splits, int m, int L, int n_heads, int head_dim, bool emit) {
  Scratch s;
  const size_t hm = (size_t)n_heads * m;
  const size_t n_blk = (size_t)(L + kBlockKeys - 1) / kBlockKeys;
  s.o_part = n_splits > 1 ? (size_t)n_splits * hm * head_dim : 0;
  s.ml = (size_t)n_splits * hm * 2;
  s.ptilde = emit ? (hm * (n_blk * kBlockKeys + kPtildePad) + 1) / 2 : 0;
  s.ptilde = (s.ptilde + 3) & ~(size_t)3;                          // keep what follows 16-byte aligned
  s.refblk = emit ? hm * n_blk : 0;
  s.total = s.o_part + s.ml + s.ptilde + s.refblk;
  return s;
}

template <int DH>
hipError_t launch_tiled(const Tunables& t, const TiledCall* calls, int n_calls, int n_heads, int n_kv_heads,
                        float* scratch, size_t scratch_floats, hipStream_t st) {
  const FwdPlan shape = plan_fwd(t, calls, n_calls, n_heads, DH);      // one for the batch
  const int q_per_wg = shape.q_per_wg();
  bool emit = false;
  for (int i = 0; i < n_calls; ++i) emit = emit || calls[i].attn_avg != nullptr;
  const float scale = 1.0f / sqrtf((float)DH);
  BatchArgs args;
  memset(&args, 0, sizeof(args));
  size_t used = 0;
  int max_tiles = 0, max_fin = 0;
  bool dma = true;                       // straight into LDS: whole 16-byte pieces, 32-bit offsets
  for (int i = 0; i < n_calls; ++i) {
    const TiledCall& c = calls[i];
    dma = dma && ((uintptr_t)c.k_cache | (uintptr_t)c.v_cache) % 16 == 0 && (size_t)c.L * n_kv_heads * DH * 2 < (1ull << 31);
    const int q_blocks = (c.m + q_per_wg - 1) / q_per_wg;
    const int blocks = (c.L + kBlockKeys - 1) / kBlockKeys;
    const int s_i = may_split(t, c.m, n_heads) ? std::max(1, std::min(shape.splits, blocks)) : 1;
    const int keys_per_split = ((blocks + s_i - 1) / s_i) * kBlockKeys;
    const int n_splits = (c.L + keys_per_split - 1) / keys_per_split;      // every split holds at least one key
    const bool emit_i = c.attn_avg != nullptr;
    const Scratch sc = scratch_of(n_splits, c.m, c.L, n_heads, DH, emit_i);
    if (sc.total > 0 && (!scratch || used + sc.total > scratch_floats)) return hipErrorInvalidValue;
    float* base = scratch ? scratch + used : nullptr;
    used += (sc.total + 3) & ~(size_t)3;
    SeqArgs& a = args.seq[i];
    a.q = (const bf16*)c.q; a.k_cache = (const bf16*)c.k_cache; a.v_cache = (const bf16*)c.v_cache;
    a.out = (bf16*)c.out; a.lse = c.lse; a.attn_avg = c.attn_avg;
    a.o_part = base;                                               // 16-byte aligned pieces, in this order
    a.ptilde = reinterpret_cast<bf16*>(base && emit_i ? base + sc.o_part : nullptr);
    a.ml_part = base ? base + sc.o_part + sc.ptilde : nullptr;
    a.refblk = base && emit_i ? a.ml_part + sc.ml : nullptr;
    a.m = c.m; a.L = c.L; a.keys_per_split = keys_per_split; a.n_splits = n_splits; a.q_blocks = q_blocks;
    a.avg_blocks = emit_i ? ((c.m + kFinRows - 1) / kFinRows) * ((blocks * kBlockKeys + kFinKeys - 1) / kFinKeys) : 0;
    const int groups = (n_heads * n_splits + 7) / 8;
    max_tiles = std::max(max_tiles, groups * 8 * q_blocks);
    const size_t items = (size_t)n_heads * c.m * (DH / 4);
    const int merge_blocks = n_splits > 1 ? (int)((items + kThreads - 1) / kThreads) : 0;
    max_fin = std::max(max_fin, a.avg_blocks + merge_blocks);
  }
  const dim3 grid(max_tiles, n_calls);
#define D2C_TILED_FWD(QT_, WAVES_, EMIT_)                                                                              \
  do {                                                                                                                 \
    if (dma)                                                                                                           \
      hipLaunchKernelGGL((attn_tiled_fwd_kernel<DH, QT_, WAVES_, EMIT_, true>), grid, dim3(WAVES_ * 64), 0, st, args,  \
                         n_heads, n_kv_heads, scale);                                                                  \
    else                                                                                                               \
      hipLaunchKernelGGL((attn_tiled_fwd_kernel<DH, QT_, WAVES_, EMIT_, false>), grid, dim3(WAVES_ * 64), 0, st, args, \
                         n_heads, n_kv_heads, scale);                                                                  \
  } while (0)
  if (shape.qt == 2 && shape.waves == 8 && emit) D2C_TILED_FWD(2, 8, true);
  else if (shape.qt == 2 && shape.waves == 8) D2C_TILED_FWD(2, 8, false);
  else if (shape.qt == 2 && emit) D2C_TILED_FWD(2, 4, true);
  else if (shape.qt == 2) D2C_TILED_FWD(2, 4, false);
  else if (shape.waves == 8) return hipErrorInvalidValue;
  else if (emit) D2C_TILED_FWD(1, 4, true);
  else D2C_TILED_FWD(1, 4, false);
#undef D2C_TILED_FWD
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || max_fin == 0) return e;
  hipLaunchKernelGGL(attn_finish_kernel<DH>, dim3((unsigned)max_fin, n_calls), dim3(kThreads), 0, st, args, n_heads);
  return hipGetLastError();
}

}  // namespace

// Most scratch ONE sequence of a batch can need, over every (m <= max_m, L <= max_L), with the head average
// wanted.  The split count follows the whole batch, so a sequence counts as split wherever it may be.
size_t attention_tiled_scratch_floats(const Tunables& t, int max_m, int max_L, int n_heads, int head_dim) {
  size_t worst = 0;
  const int max_splits = std::max(1, std::min(8, t.attn_max_splits));
  for (int L = kBlockKeys;; L += kBlockKeys) {
    const int Lc = std::min(L, max_L);
    const int blocks = (Lc + kBlockKeys - 1) / kBlockKeys;
    for (int m = 1; m <= max_m; ++m) {
      const int n_splits = may_split(t, m, n_heads) ? std::min(max_splits, blocks) : 1;
      worst = std::max(worst, (scratch_of(n_splits, m, Lc, n_heads, head_dim, true).total + 3) & ~(size_t)3);
    }
    if (L >= max_L) break;
  }
  return worst;
}

hipError_t launch_attention_tiled(const Tunables& t, const TiledCall* calls, int n_calls, int n_heads, int n_kv_heads,
                                  int head_dim, float* scratch, size_t scratch_floats, hipStream_t st) {
  if (n_calls <= 0) return hipSuccess;
  if (n_calls > kMaxBatch) return hipErrorInvalidValue;
  if (head_dim == 128) return launch_tiled<128>(t, calls, n_calls, n_heads, n_kv_heads, scratch, scratch_floats, st);
  if (head_dim == 64) return launch_tiled<64>(t, calls, n_calls, n_heads, n_kv_heads, scratch, scratch_floats, st);
  return hipErrorInvalidValue;
}

int attention_tiled_max_batch() { return kMaxBatch; }

}  // namespace d2c
