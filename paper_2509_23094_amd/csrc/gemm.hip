// Weight-streaming GEMM for the ragged handful of selected rows (Eq. 5 of the
// d2Cache paper feeds only the rows M* u U through the model, so every
// projection is  P = A[m,K] * W[N,K]^T  with m of the order of 100 or less).
//
// At such m the arithmetic intensity is about m FLOP per weight byte, far below
// the chip's ridge: the kernel is bound by streaming W from HBM once.  Design:
//   * each wave owns 16*NT weight rows (output columns) and reads them straight
//     from global memory into matrix-core operand registers, 16 bytes per lane,
//     256 contiguous bytes per weight row and chunk, through a register ring that
//     keeps RING-1 chunks in flight ahead of the one being consumed (row-major
//     weights come through LDS instead, see kRowStaged);
//   * the activation rows (shared by all waves of the workgroup) are staged
//     through LDS in 256-byte-per-row chunks, double-buffered, one barrier per chunk;
//     a chunk is requested two iterations before it is needed in LDS, so its
//     latency never sits between two barriers;
//   * the contraction axis can be split over several workgroups; every split writes
//     its own fp32 partial and the consumer kernel sums the partials in a fixed order
//     (deterministic, no atomics);
//   * more than 128 rows are covered by several row chunks (many rows in bf16: NT = 4, or gemm_wide_kernel below).
//     The grid is one-dimensional and workgroup ids are dealt round-robin to the 8
//     XCDs, each with its own L2: the mapping below gives the row chunks of one weight
//     tile consecutive slots of the SAME XCD, so the tile comes from HBM once and the
//     other chunks hit it in L2.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "internal.h"

namespace d2c {

namespace {

constexpr int kChunkBytes = 256;                 // bytes of one row in one chunk
constexpr int kRowStride = kChunkBytes + 16;     // LDS row pitch: 16-byte skew, conflict-free 16-byte reads
constexpr int kSteps = 4;                        // matrix-core steps per chunk
constexpr int kSuperRows = 8, kSuperCols = 4;    // many rows: block of workgroups that share an XCD's L2

// RING = number of weight chunks a wave keeps in registers (one being consumed, RING-1 in flight).
// MODE: 0 = W row-major [N, K]; 1 = W pre-tiled; 2 = W pre-tiled with gate and up tiles interleaved and the
// SwiGLU applied in the epilogue (single k split, one column tile per wave): act[m, N/2] = T(silu(g) * u).
// 3 = W row-major, its rows staged through LDS (16-byte aligned rows, one column tile per wave, where LDS holds it).
enum { kRowMajor = 0, kPre = 1, kPreSwiglu = 2, kRowStaged = 3 };
// weight chunks of a wave in LDS, one in use and the others on their way: 3, or 2 where three do not fit; 0 = neither
template <int MT, int NT, int WAVES>
constexpr int kStageSlots = NT != 1 ? 0
                            : 2 * MT * 16 * kRowStride + WAVES * 3 * 16 * kChunkBytes <= 160 * 1024 ? 3
                            : 2 * MT * 16 * kRowStride + WAVES * 2 * 16 * kChunkBytes <= 160 * 1024 ? 2
                                                                                                     : 0;

// silu(g) * u with the quotient from the reciprocal unit and one correction from its own remainder (Markstein's method), as
// exact as the division that it replaces: relative error against 64 bits over |g| < 16 at most 1.5e-7, 4e-8 on average, both.
// The exponential unit alone (arguments rounded after the product with log2(e)) reaches 1e-6 and is not used.
__device__ __forceinline__ float gate_of(float g, float e, float u) {      // e = exp(-g), finite
  const float d = 1.0f + e, inv = __builtin_amdgcn_rcpf(d), q = g * inv;
  return copysignf(fmaf(fmaf(-d, q, g), inv, q), g) * u;       // the correction of -0 would lose its sign
}
__device__ __forceinline__ float gated(float g, float u) {
  if (!(fabsf(g) < 87.0f)) return g / (1.0f + expf(-g)) * u;   // the steps above need finite terms
  return gate_of(g, expf(-g), u);
}
// Four values of a lane.  Where all gates of the wave are finite and below 87 this is one stretch of code without branches, which
// overlaps their latencies.  Both sides give an ordinary gate the same bits: a value depends on its own gate alone.
__device__ __forceinline__ f32x4 gated4(const f32x4& g, const f32x4& u) {
  bool wide = false;
#pragma unroll
  for (int j = 0; j < 4; ++j) wide = wide || !(fabsf(g[j]) < 87.0f);
  f32x4 o;
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(wide) != 0, 0)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = gated(g[j], u[j]);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = gate_of(g[j], expf(-g[j]), u[j]);
  }
  return o;
}

template <typename T, int MT, int NT, int WAVES, int MODE>
__global__ __launch_bounds__(WAVES * 64) void gemm_rows_kernel(
    const T* __restrict__ A, int lda, const T* __restrict__ W, int ldw, float* __restrict__ P, int ldp,
    size_t split_stride, int m, int N, int K, int k_per_split, int n_blocks, int n_splits, int row_chunks, int rot_mul,
    T* __restrict__ act) {
  constexpr bool PRE = MODE == kPre || MODE == kPreSwiglu, STAGED = MODE == kRowStaged;
  static_assert(!STAGED || kStageSlots<MT, NT, WAVES> != 0, "staged weights must fit LDS");
  static_assert(MODE != kPreSwiglu || NT % 2 == 0 || WAVES % 2 == 0, "the SwiGLU epilogue pairs neighbouring waves");
  constexpr int RING = 2;
  constexpr int kThreads = WAVES * 64;
  constexpr int kAFrags = MT * 256;                              // 16-byte fragments of one activation chunk
  constexpr int AI = (kAFrags + kThreads - 1) / kThreads;        // of which one thread moves this many
  // workgroup id -> (weight tile, row chunk): id % 8 is the XCD, within an XCD the row chunk varies fastest
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  int tile, bz;
  if constexpr (NT >= 4) {
    // Many rows: the 32 workgroups that run on an XCD at one time form a block of kSuperRows row chunks x
    // kSuperCols weight tiles, so that what its L2 has to bring in per k-step (8 x 128 activation rows +
    // 4 x 256 weight rows) is less than half of that of 32 row chunks of one weight tile.
    const int n_row_st = (row_chunks + kSuperRows - 1) / kSuperRows;
    const int st = slot / (kSuperRows * kSuperCols), w = slot % (kSuperRows * kSuperCols);
    bz = (st % n_row_st) * kSuperRows + w % kSuperRows;
    tile = ((st / n_row_st) * kSuperCols + w / kSuperRows) * 8 + xcd;
    if (bz >= row_chunks) return;
  } else {
    tile = (slot / row_chunks) * 8 + xcd;
    bz = slot % row_chunks;
  }
  if (tile >= n_blocks * n_splits) return;       // padding (whole workgroup leaves)
  const int by = tile / n_blocks, bx = tile - by * n_blocks;
  constexpr int E = Frag<T>::kElems;
  constexpr int KS = Frag<T>::kStep;
  constexpr int KC = kSteps * KS;                // elements per chunk (= 256 bytes)
  constexpr int PB = RING - 1;                   // prefetch distance of the weight stream, in chunks
  __shared__ __attribute__((aligned(16))) unsigned char lds[2][MT * 16 * kRowStride];

  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  const int row0 = bz * (MT * 16);
  const int k_begin = by * k_per_split;
  const int k_end = min(K, k_begin + k_per_split);
  const int n_base = (bx * WAVES + wave) * (16 * NT);
  const int n_chunks = (k_end - k_begin + KC - 1) / KC;

  // this lane's weight rows (clamped: out-of-range columns are computed on a valid row and dropped).
  // PRE: W is the pre-tiled copy (see preshuffle_kernel): [16-row tile][256-byte chunk][step][lane][16 B],
  // ldw = chunks per tile; wrow then points at this lane's 16 bytes of step 0 of the tile's chunk 0.
  constexpr int kBlockElems = 16 * KC;           // elements of one 16-row x 256-byte block (4 KB)
  const T* wrow[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    if (PRE) {
      const int t16 = min((n_base + nt * 16) / 16, (N + 15) / 16 - 1);
      wrow[nt] = W + (size_t)t16 * ldw * kBlockElems + lane * E;
    } else {
      int n = min(n_base + nt * 16 + r, N - 1);
      wrow[nt] = W + (size_t)n * ldw;
    }
  }

  Frag<T> areg[2][AI];                 // areg[c & 1]: activation chunk c on its way from global memory to LDS
  Frag<T> breg[RING][NT][kSteps];      // breg[c % RING]: weight chunk c
  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

  // The loop below has no conditional loads or stores.  A load under a branch makes the compiler wait
  // for ALL outstanding loads before the next use, which would drain the prefetch ring every iteration;
  // so addresses are clamped instead: rows >= m read row m-1 (their accumulators are never stored),
  // chunks past the end re-read the last chunk (an L2 hit, never used), and the weight fragments of the
  // last chunk's tail are masked to zero where they are consumed.
  const int last_row = m - 1;
  const int last_chunk = n_chunks - 1;
  // Workgroups walk their k-range from different starting chunks (a rotation by a multiple of the
  // column-block index), so that at one moment they do not all ask for the same offsets within a row.
  const int rot = n_chunks > 0 ? (int)(((unsigned)bx * (unsigned)rot_mul) % (unsigned)n_chunks) : 0;
  auto chunk_k = [&](int chunk) {
    int p = min(chunk, last_chunk) + rot;
    if (p >= n_chunks) p -= n_chunks;
    return k_begin + p * KC;
  };
  auto load_a = [&](Frag<T> (&a)[AI], int chunk) {
    const int kc = chunk_k(chunk);
#pragma unroll
    for (int i = 0; i < AI; ++i) {
      // fragment id in the chunk: row f/16, 16-byte column f%16; ids past the end repeat the last one
      const int f = min(tid + i * kThreads, kAFrags - 1);
      const int row = min(row0 + (f >> 4), last_row);
      const int k = min(kc + (f & 15) * E, k_end - E);
      a[i].raw = ld16(A + (size_t)row * lda + k);
    }
  };
  auto store_a = [&](const Frag<T> (&a)[AI], int buf) {
#pragma unroll
    for (int i = 0; i < AI; ++i) {
      const int f = min(tid + i * kThreads, kAFrags - 1);
      *reinterpret_cast<u32x4*>(&lds[buf][(f >> 4) * kRowStride + (f & 15) * 16]) = a[i].raw;
    }
  };
  // One column tile per wave means one row chunk: every weight byte is read by exactly one workgroup of the
  // launch, so its loads carry the streaming hint and leave the L2 to the activations and partial sums.
  auto ldw16 = [](const T* p) {
    if constexpr (NT == 1) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    else return ld16(p);
  };
  auto load_b = [&](Frag<T> (&b)[NT][kSteps], int chunk) {
    const int kc = chunk_k(chunk);
    if (PRE) {
      // one instruction = 1 KB contiguous: whole cache lines, no clamping (the copy is zero-padded)
      const size_t off = (size_t)(kc / KC) * kBlockElems;
#pragma unroll
      for (int s = 0; s < kSteps; ++s)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) b[nt][s].raw = ldw16(wrow[nt] + off + s * 64 * E);
    } else {
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        const int k = min(kc + s * KS + g * E, k_end - E);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) b[nt][s].raw = ldw16(wrow[nt] + k);
      }
    }
  };

  // The products of one chunk: activation fragments from LDS, b_of(step, column tile) the weights.  In bf16 from 2 row tiles on
  // the fragments are read kAhead of them ahead of their use and the scheduler is told to keep it so: left alone it waits for each
  // read in front of its step, with 7 row tiles 28 LDS latencies a chunk, longer than the chunk's weights take (97 rows x 3584 x
  // 18944 38.8 -> 33 us, x 37888 x 3584 66 -> 57, x 4608 x 3584 13.3 -> 12.4; 128 x 24576 x 4096 60 -> 54; 200, two column tiles a
  // wave, 78 -> 71; 69 rows 3 %, 46 rows 1 %; one row tile loses: 16 x 152064 x 3584 180 -> 184).  A barrier for the scheduler
  // behind the chunk costs half of that: the next chunk's way into LDS has to start beside the last products.  Four ahead in 8 waves
  // cost the second workgroup on a compute unit its registers (112 x 126464 x 4096 229 us).  So do three with 7 and 8 row tiles (129
  // and 132 registers), which shows in the head's several rounds only (us without / three / two ahead: 112 x 126464 x 4096 214 / 216 /
  // 210, 128 rows 218 / 221 / 225; x 152064 x 3584 243.6 / 242.8 / 237.5 and 251.1 / 250.5 / 255.5), while a layer's single rounds
  // gain (LLaDA layer of 112 rows 152.6 / 146.8 / 148.7, of 128 159 / 153 / 155.6).
  auto chunk_steps = [&](const unsigned char* abuf, auto b_of) {
    auto read_af = [&](int i) {
      Frag<T> f;
      f.raw = *reinterpret_cast<const u32x4*>(&abuf[((i % MT) * 16 + r) * kRowStride + ((i / MT) * 4 + g) * 16]);
      return f;
    };
    constexpr int NI = kSteps * MT;
    if constexpr (sizeof(T) == 2 && MT >= 2) {
      constexpr int kAhead = WAVES == 8 || WAVES == 6 ? 3 : 4;
      Frag<T> af[kAhead], bf[NT];
#pragma unroll
      for (int i = 0; i < kAhead; ++i) af[i] = read_af(i);
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        if (i % MT == 0) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) bf[nt] = b_of(i / MT, nt);
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) mfma16(acc[i % MT][nt], af[i % kAhead], bf[nt]);
        if (i + kAhead < NI) af[i % kAhead] = read_af(i + kAhead);
      }
      __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);
        if (i + kAhead < NI) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    } else {
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        Frag<T> bf[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) bf[nt] = b_of(s, nt);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const Frag<T> af = read_af(s * MT + mt);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) mfma16(acc[mt][nt], af, bf[nt]);
        }
      }
    }
  };

  if (n_chunks <= 0) return;
  if constexpr (NT >= 4) {
    // Many rows: 128 x 64 outputs per wave, one wave per SIMD.  Nothing else hides latencies here, so the
    // loop is pipelined by hand and the scheduler is told to keep the interleaving:
    //   * the activation fragments are read from LDS three matrix-core groups ahead of their use;
    //   * the weight registers of a k-step are refilled as soon as that step is done, with the same step
    //     of the chunk two ahead (two chunks of flight time: an L2 miss costs more than one);
    //   * the next activation chunk is requested at the top of an iteration and stored behind it.
    // The launcher guarantees whole chunks and an even number of them per split: nothing to mask.
    static_assert(RING == 2, "the wide loop keeps two weight chunks");
    constexpr int NI = kSteps * MT;
    auto load_b_step = [&](Frag<T> (&b)[NT][kSteps], int chunk, int step) {
      const size_t off = PRE ? (size_t)(chunk_k(chunk) / KC) * kBlockElems + step * 64 * E
                             : (size_t)(chunk_k(chunk) + step * KS + g * E);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) b[nt][step].raw = ld16(wrow[nt] + off);
    };
    load_a(areg[0], 0);
    load_b(breg[0], 0);
    load_b(breg[1], 1);
    store_a(areg[0], 0);
    __syncthreads();
    for (int base = 0; base < n_chunks; base += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = base + u;
        load_a(areg[0], c + 1);
        __builtin_amdgcn_sched_barrier(0);
        const unsigned char* abuf = lds[u];
        auto read_af = [&](int i) {
          Frag<T> f;
          f.raw = *reinterpret_cast<const u32x4*>(&abuf[((i % MT) * 16 + r) * kRowStride + ((i / MT) * 4 + g) * 16]);
          return f;
        };
        Frag<T> af[4];
        af[0] = read_af(0);
        af[1] = read_af(1);
        af[2] = read_af(2);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) mfma16(acc[i % MT][nt], af[i % 4], breg[u][nt][i / MT]);
          if (i + 3 < NI) af[(i + 3) % 4] = read_af(i + 3);
          if (i % MT == MT - 1) load_b_step(breg[u], c + 2, i / MT);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);                          // NT matrix-core instructions
          if (i + 3 < NI) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);           // one LDS read
          if (i % MT == MT - 1) __builtin_amdgcn_sched_group_barrier(0x020, NT, 0);    // the k-step's refill
        }
        __builtin_amdgcn_sched_barrier(0);
        store_a(areg[0], u ^ 1);
        __syncthreads();
      }
    }
  } else if constexpr (STAGED) {
    // Row-major weights in operand order (lane = row) cost the L1, which merges only what consecutive lanes ask for, 64
    // accesses an instruction.  A wave therefore brings its 16 rows straight into LDS, four whole 256-byte row pieces an
    // instruction, up to two chunks ahead, and reads its operands there (the 16-byte pieces of a row are xored with its number:
    // eight lanes of a read touch different banks).  Nobody else reads them: no barrier, but the wave's own wait.
    // LLaDA shapes: the head on 17 rows (126464 x 4096) 242 -> 210 us, gate/up on 46 rows 49 -> 40, QKV 32 -> 27.
    constexpr int SL = kStageSlots<MT, NT, WAVES>;
    __shared__ __attribute__((aligned(16))) unsigned char wst[WAVES * SL * 16 * kChunkBytes];
    unsigned char* const mine = wst + __builtin_amdgcn_readfirstlane(wave) * (SL * 16 * kChunkBytes);
    const int first = min(__builtin_amdgcn_readfirstlane(n_base), N - 1), rows_left = N - 1 - first;
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(W) + (size_t)first * ldw, 0, (int)(((size_t)min(15, rows_left) * ldw + K) * sizeof(T)), 0x00020000);
    int roff[4], poff[4];                                  // instruction i: row 4 i + lane / 16, its piece of the chunk
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = i * 4 + (lane >> 4);
      roff[i] = (int)(min(row, rows_left) * (size_t)ldw * sizeof(T));
      poff[i] = ((lane & 15) ^ (row & 7)) * E;
    }
    const uint32_t mine_at = lds_address(mine);
    uint32_t woff[kSteps];                                 // this lane's operand of step s inside a slot
#pragma unroll
    for (int s = 0; s < kSteps; ++s) woff[s] = (uint32_t)(r * kChunkBytes + ((s * 4 + g) ^ (r & 7)) * 16);
    auto stage_w = [&](int chunk, int slot) {
      const int kc = chunk_k(chunk);
#pragma unroll
      for (int i = 0; i < 4; ++i)                          // pieces past the end repeat the last one and meet zeros
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            wrsrc, (__attribute__((address_space(3))) void*)(mine + slot * (16 * kChunkBytes) + i * 1024), 16,
            roff[i] + min(kc + poff[i], k_end - E) * (int)sizeof(T), 0, 0, 2 /* streaming */);
    };
    auto fence = [] {
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    load_a(areg[0], 0);
    fence();
    stage_w(0, 0);
    fence();
    load_a(areg[1], 1);
    fence();
#pragma unroll
    for (int p = 1; p + 1 < SL; ++p) stage_w(p, p);
    fence();
    store_a(areg[0], 0);
    __syncthreads();
    int slot = 0;
    for (int base = 0; base < n_chunks; base += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = base + u;
        const int refill = slot == 0 ? SL - 1 : slot - 1;  // consumed by the iteration before
        load_a(areg[u & 1], c + 2);
        fence();
        stage_w(c + SL - 1, refill);
        fence();
        // this chunk's rows have arrived: requested behind them were SL - 1 stagings and as many activation chunks
        constexpr int kVm = (SL - 1) * (AI + 4);
        static_assert(kVm < 64, "vmcnt has 6 bits");
        __builtin_amdgcn_s_waitcnt((kVm & 15) | ((kVm >> 4) << 14) | 0x70 | 0xf00);
        fence();
        const unsigned char* abuf = lds[u & 1];
        const uint32_t wbuf = mine_at + (uint32_t)(slot * (16 * kChunkBytes));
        const int kc = chunk_k(c);
        u32x4 wv[kSteps];
        lds_read_staged(wv, wbuf + woff[0], wbuf + woff[1], wbuf + woff[2], wbuf + woff[3]);
        chunk_steps(abuf, [&](int s, int) {
          const unsigned keep = (c < n_chunks && kc + s * KS + g * E < k_end) ? 0xffffffffu : 0u;
          Frag<T> bf;
          bf.raw = wv[s] & u32x4{keep, keep, keep, keep};
          return bf;
        });
        fence();
        store_a(areg[(u + 1) & 1], (u + 1) & 1);
        __builtin_amdgcn_s_waitcnt(0xc07f);                // lgkmcnt(0): the stores; what is on its way stays so
        fence();
        __builtin_amdgcn_s_barrier();
        fence();
        slot = slot == SL - 1 ? 0 : slot + 1;
      }
    }
    __builtin_amdgcn_s_waitcnt(0x70 | 0xf00);              // no staging may write LDS after the workgroup has left
  } else {
  // prologue: weight chunks 0..PB-1 and activation chunks 0, 1 are requested; chunk 0 reaches LDS
#pragma unroll
  for (int u = 0; u < PB; ++u) load_b(breg[u], u);
  load_a(areg[0], 0);
  load_a(areg[1], 1);
  store_a(areg[0], 0);
  __syncthreads();

  for (int base = 0; base < n_chunks; base += RING) {
#pragma unroll
    for (int u = 0; u < RING; ++u) {
      // no early exit: iterations past the last chunk (at most RING-1) re-read it and contribute zero,
      // which keeps the RING iterations one basic block that the scheduler can interleave freely
      const int c = base + u;
      // requests first: activation chunk c+2 (its registers were emptied into LDS one iteration ago)
      // and weight chunk c+PB
      load_a(areg[u & 1], c + 2);
      load_b(breg[(u + PB) % RING], c + PB);
      __builtin_amdgcn_sched_barrier(0);   // the requests stay ahead of this iteration's arithmetic
      const unsigned char* abuf = lds[u & 1];
      const int kc = chunk_k(c);
      chunk_steps(abuf, [&](int s, int nt) {     // zero in the tail of the last chunk and past it
        const unsigned keep = (c < n_chunks && kc + s * KS + g * E < k_end) ? 0xffffffffu : 0u;
        Frag<T> bf;
        bf.raw = breg[u][nt][s].raw & u32x4{keep, keep, keep, keep};
        return bf;
      });
      // activation chunk c+1 was requested one iteration ago: its latency is behind us
      store_a(areg[(u + 1) & 1], (u + 1) & 1);
      __syncthreads();
    }
  }
  }   // weights through registers

  if (MODE == kPreSwiglu && NT % 2 == 0) {
    // Column tiles alternate gate, up, gate, up ..: with an even number of tiles per wave each pair sits in one wave
    const int F = N >> 1;
#pragma unroll
    for (int p = 0; p < NT / 2; ++p) {
      const int col = ((n_base >> 5) + p) * 16 + r;             // n_base = 32 * (first hidden tile of the wave)
      if (col >= F) continue;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int row = row0 + mt * 16 + g * 4 + j;
          const float gv = acc[mt][2 * p][j];
          if (row < m)
            act[(size_t)row * F + col] = from_f32<T>(gv / (1.0f + expf(-gv)) * acc[mt][NT > 1 ? 2 * p + 1 : 0][j]);
        }
    }
    return;
  }
  if (MODE == kPreSwiglu) {
    // Column tiles alternate gate, up, gate, up ..: wave 2p holds the gate values and wave 2p+1 the up
    // values of the same 16 hidden columns.  The odd wave hands its accumulators over through LDS (the
    // activation buffers are idle: the loop ended on a barrier), the even wave applies the gate.
    f32x4* xch = reinterpret_cast<f32x4*>(&lds[0][0]);          // [WAVES/2][MT][64]
    const int pair = wave >> 1;
    if (wave & 1) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xch[(pair * MT + mt) * 64 + lane] = acc[mt][0];
    }
    __syncthreads();
    if (wave & 1) return;
    const int F = N >> 1;
    const int col = (n_base >> 5) * 16 + r;                     // n_base = 32 * (hidden tile)
    if (col >= F) return;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const f32x4 u = xch[(pair * MT + mt) * 64 + lane];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = row0 + mt * 16 + g * 4 + j;
        const float gv = acc[mt][0][j];
        if (row < m) act[(size_t)row * F + col] = from_f32<T>(gv / (1.0f + expf(-gv)) * u[j]);
      }
    }
    return;
  }
  float* out = P + (size_t)by * split_stride;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int col = n_base + nt * 16 + r;
      if (col >= N) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = row0 + mt * 16 + g * 4 + j;
        if (row < m) out[(size_t)row * ldp + col] = acc[mt][nt][j];
      }
    }
}

// ---- many rows (bf16): two row chunks of 16*MT rows x 256 columns per workgroup.  8 waves: four take a row chunk, each with
// 64 columns, so that two waves share a SIMD (one alone cannot issue 16x16x32 steps back to back: 1.37 PFLOP/s in a loop
// of nothing else, 1.90 with two).  What bounds the loop is how much a compute unit gets through its L1, so the tile is
// as large as the registers take (128 accumulators a lane; 256 x 256 outputs a workgroup) and the accesses are whole
// 64-byte pieces (see the staging below).  The activations go from global memory straight into LDS, a chunk of 128 k
// ahead; the weights straight into operand registers, refilled with the next chunk's step as soon as a step is done; LDS
// reads run three matrix-core groups ahead of their use.  The scheduler is told to keep that order.  The wait in front
// of the barrier leaves the weight refills behind the staging in flight.
// 512 rows, LLaDA widths, against 128 x 256 tiles of 4 waves with activations through registers: gate/up (24576 x 4096)
// 142 -> 95 us (1.09 PFLOP/s), QKV 79 -> 52.  Tried on the 256-column tile (105 us, gate/up): 32x32x16 steps with one wave
// per SIMD (119 us), operand-order staging (130 us).  Where the workgroups are too few for the chip the other is the faster:
// see plan_gemm.
// The launcher guarantees whole chunks of k: nothing to mask.
template <int MT, int NT, int MODE>
__global__ __launch_bounds__(512, 1) void gemm_wide_kernel(const bf16* __restrict__ A, int lda, const bf16* __restrict__ W,
                                                           int ldw, float* __restrict__ P, int ldp, size_t split_stride,
                                                           int m, int N, int K, int k_per_split, int n_blocks,
                                                           int n_splits, int pairs, int rot_mul, bf16* __restrict__ act) {
  constexpr bool PRE = MODE != kRowMajor;
  constexpr int E = 8, KS = 32, KC = 128;
  constexpr int kBlockElems = 16 * KC;
  constexpr int kBuf = MT * 8 * 1024;                       // bytes of one activation chunk: 2*MT row tiles x 4 steps x 1 KB
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * kBuf];
  // workgroup id -> (weight tile, row pair): id % 8 is the XCD; the 32 workgroups that run on an XCD at one time form a
  // block of up to kSuperRows row pairs x as many weight tiles, so that its L2 brings in each byte once for several
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int rows_st = min(pairs, kSuperRows);
  const int n_row_st = (pairs + rows_st - 1) / rows_st;
  const int cols_st = 32 / rows_st;
  const int st = slot / (rows_st * cols_st), in_st = slot % (rows_st * cols_st);
  const int bz = (st % n_row_st) * rows_st + in_st % rows_st;
  const int tile = ((st / n_row_st) * cols_st + in_st / rows_st) * 8 + xcd;
  if (bz >= pairs || tile >= n_blocks * n_splits) return;      // padding (whole workgroup leaves)
  const int by = tile / n_blocks, bx = tile - by * n_blocks;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  // row chunk of the pair, 64-column quarter: the two waves of a quarter sit on different SIMDs, so that they go at one pace
  // and the second finds the weights in the L1 (on one SIMD they took turns: a third more requests to the L2)
  const int part = (wave >> 1) & 1, quarter = (wave & 1) | ((wave >> 2) << 1);
  const int row0 = (bz * 2 + part) * (MT * 16);
  const int k_begin = by * k_per_split;
  const int k_end = min(K, k_begin + k_per_split);
  const int n_base = (bx * 4 + quarter) * (16 * NT);
  const int n_chunks = (k_end - k_begin) / KC;
  if (n_chunks <= 0) return;
  const int last_chunk = n_chunks - 1;

  const bf16* wrow[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    if (PRE) {
      const int t16 = min((n_base + nt * 16) / 16, (N + 15) / 16 - 1);
      wrow[nt] = W + ((size_t)t16 * ldw + k_begin / KC) * kBlockElems + lane * E;
    } else {
      wrow[nt] = W + (size_t)min(n_base + nt * 16 + r, N - 1) * ldw + k_begin + g * E;
    }
  }
  // staging: a wave brings k-step `quarter` of every other 16-row tile, 16 rows x 64 bytes an instruction (rows past m
  // repeat row m-1 and are not stored).  Four neighbouring lanes take the 64 bytes of one row: the L1 merges only what
  // consecutive lanes ask for, and operand order (lane = row) would cost it 64 accesses an instruction instead of 16.
  // LDS then holds [row][piece], the pieces of a row xored with half its number: eight lanes of an operand read (rows at one
  // k group) then touch 128 different bytes' banks.
  unsigned aoff[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
    aoff[i] = (unsigned)(((size_t)min(bz * (MT * 32) + (2 * i + part) * 16 + (lane >> 2), m - 1) * lda + quarter * KS +
                          ((lane & 3) ^ (lane >> 3 & 3)) * E) * 2);
  // (through a buffer resource: a global_load .. lds counts as a flat access, behind which every LDS wait drains the queue)
  const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16*>(A), 0, (int)(unsigned)(((size_t)(m - 1) * lda + K) * 2), 0x00020000);

  Frag<bf16> b[NT][kSteps];
  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto stage = [&](int buf, int chunk) {
    const int soff = (k_begin + chunk * KC) * 2;
#pragma unroll
    for (int i = 0; i < MT; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          arsrc, (__attribute__((address_space(3))) void*)(lds + buf * kBuf + ((2 * i + part) * 4 + quarter) * 1024), 16, (int)aoff[i],
          soff, 0, 0);
  };
  auto load_b_step = [&](int chunk, int step) {
    const size_t off = (size_t)chunk * (PRE ? kBlockElems : KC) + step * (PRE ? 64 * E : KS);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) b[nt][step].raw = ld16(wrow[nt] + off);
  };
  // the walk over the chunks starts at a multiple of the column block, as in the rows kernel; behind the last chunk it
  // requests that one again (an L2 hit, never used)
  int at = (int)(((unsigned)bx * (unsigned)rot_mul) % (unsigned)n_chunks);
  stage(0, at);
#pragma unroll
  for (int s = 0; s < kSteps; ++s) load_b_step(at, s);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x70 | 0xf00);                  // vmcnt(0)
  __syncthreads();
  constexpr int NI = kSteps * MT;
  for (int c = 0; c < n_chunks; ++c) {
    if (c < last_chunk) at = at == last_chunk ? 0 : at + 1;
    stage((c & 1) ^ 1, at);
    __builtin_amdgcn_sched_barrier(0);
    const unsigned char* abuf = lds + (c & 1) * kBuf + part * (MT * 4096) + (r * 4 + (g ^ (r >> 1 & 3))) * 16;
    auto read_af = [&](int i) {
      Frag<bf16> f;
      f.raw = *reinterpret_cast<const u32x4*>(abuf + ((i % MT) * 4 + i / MT) * 1024);
      return f;
    };
    Frag<bf16> af[4];
    af[0] = read_af(0);
    af[1] = read_af(1);
    af[2] = read_af(2);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) mfma16(acc[i % MT][nt], af[i % 4], b[nt][i / MT]);
      if (i + 3 < NI) af[(i + 3) % 4] = read_af(i + 3);
      if (i % MT == MT - 1) load_b_step(at, i / MT);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);                          // NT matrix-core instructions
      if (i + 3 < NI) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);           // one LDS read
      if (i % MT == MT - 1) __builtin_amdgcn_sched_group_barrier(0x020, NT, 0);    // the k-step's refill
    }
    __builtin_amdgcn_sched_barrier(0);
    // the next chunk is in LDS once all but the weight refills requested behind its staging has arrived
    constexpr int kVm = 4 * NT;
    __builtin_amdgcn_s_waitcnt((kVm & 15) | ((kVm >> 4) << 14) | 0x70 | 0xf00);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_s_waitcnt(0x70 | 0xf00);                  // no staging may write LDS after the workgroup has left

  if constexpr (MODE == kPreSwiglu) {
    // column tiles alternate gate, up, gate, up ..  The gated values go through LDS (idle now) and out in 16-byte pieces of
    // rows: 2-byte stores from the accumulators, with a branch for each, took 5-8 us of the kernel (rows x 24576 x 4096, fastest
    // of 40 launches, the 2 % of the waves' order included: 860 rows 159 -> 151 us, 512 rows 91.6 -> 87.4; steps of many rows 3 %).
    constexpr int kCols = 32 * NT, kPitch = kCols + 8;        // hidden columns of the workgroup
    constexpr int kXch = NT % 2 == 0 ? 0 : 4 * MT * 1024;
    static_assert(kXch + 2 * MT * 16 * kPitch * 2 <= 2 * kBuf, "the output tile and the exchanged tiles fit the staging buffers");
    const int F = N >> 1;
    bf16* const tile = reinterpret_cast<bf16*>(lds + kXch);
    auto put = [&](int pair, int mt, const f32x4& gate, const f32x4& up) {      // pair: of the workgroup's
      const f32x4 o = gated4(gate, up);
      bf16* dst = tile + (part * (MT * 16) + mt * 16 + g * 4) * kPitch + pair * 16 + r;
#pragma unroll
      for (int j = 0; j < 4; ++j) dst[j * kPitch] = (bf16)o[j];
    };
    __syncthreads();
    if constexpr (NT % 2 == 0) {                              // every pair sits in one wave
#pragma unroll
      for (int p = 0; p < NT / 2; ++p)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) put(quarter * (NT / 2) + p, mt, acc[mt][2 * p], acc[mt][2 * p + 1]);
    } else {
      // three tiles: an even quarter holds a pair and the gate tile of another, whose up tile is its neighbour's first; they
      // exchange halves of these two tiles.  The neighbour's other two are a pair of their own.
      static_assert(NT == 3, "pairs across two waves");
      constexpr int kHalf = MT / 2;
      f32x4* xch = reinterpret_cast<f32x4*>(lds) + (part * 2 + (quarter >> 1)) * (MT * 64);      // [MT][64]
      const int first = (quarter >> 1) * 3;
      const bool odd = quarter & 1;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        if (odd == (mt < kHalf)) xch[mt * 64 + lane] = odd ? acc[mt][0] : acc[mt][2];
      __syncthreads();
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        if (odd) put(first + 2, mt, acc[mt][1], acc[mt][2]);
        else put(first, mt, acc[mt][0], acc[mt][1]);
        if (odd != (mt < kHalf)) {
          const f32x4 other = xch[mt * 64 + lane];
          put(first + 1, mt, odd ? other : acc[mt][2], odd ? acc[mt][0] : other);
        }
      }
    }
    __syncthreads();
    constexpr int kPieces = kCols / 8;
    for (int i = tid; i < 2 * MT * 16 * kPieces; i += 512) {
      const int row_t = i / kPieces, piece = i - row_t * kPieces;
      const int row = bz * (MT * 32) + row_t, col = bx * kCols + piece * 8;
      if (row < m && col < F)
        *reinterpret_cast<u32x4*>(act + (size_t)row * F + col) = *reinterpret_cast<const u32x4*>(tile + row_t * kPitch + piece * 8);
    }
    return;
  }
  float* out = P + (size_t)by * split_stride;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int col = n_base + nt * 16 + r;
      if (col >= N) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = row0 + mt * 16 + g * 4 + j;
        if (row < m) out[(size_t)row * ldp + col] = acc[mt][nt][j];
      }
    }
}

template <int MT, int NT, int MODE>
hipError_t launch_wide_t(const GemmPlan& pl, int pairs, const void* A, int lda, const void* W, int ldw, float* P, int ldp,
                         size_t split_stride, int m, int N, int K, hipStream_t st, void* act) {
  const int n_blocks = (N + 64 * NT - 1) / (64 * NT);
  const int groups = (n_blocks * pl.splits + 7) / 8;            // weight tiles are dealt to the XCDs in groups of 8
  const int rows_st = pairs < kSuperRows ? pairs : kSuperRows;
  const int cols_st = 32 / rows_st;
  const dim3 grid(8 * ((groups + cols_st - 1) / cols_st) * ((pairs + rows_st - 1) / rows_st) * (rows_st * cols_st));
  hipLaunchKernelGGL((gemm_wide_kernel<MT, NT, MODE>), grid, dim3(512), 0, st, (const bf16*)A, lda, (const bf16*)W, ldw, P,
                     ldp, split_stride, m, N, K, pl.k_per_split, n_blocks, pl.splits, pairs, pl.rot, (bf16*)act);
  return hipGetLastError();
}
template <int MODE>
hipError_t launch_wide(const GemmPlan& pl, const void* A, int lda, const void* W, int ldw, float* P, int ldp,
                       size_t split_stride, int m, int N, int K, hipStream_t st, void* act) {
  const int pairs = (pl.row_chunks + 1) / 2;
#define D2C_WIDE(mt_)                                                                                                        \
  if (pl.mt == mt_ && (pl.nt == 3 || pl.nt == 4))                                                                            \
    return pl.nt == 3 ? launch_wide_t<mt_, 3, MODE>(pl, pairs, A, lda, W, ldw, P, ldp, split_stride, m, N, K, st, act)       \
                      : launch_wide_t<mt_, 4, MODE>(pl, pairs, A, lda, W, ldw, P, ldp, split_stride, m, N, K, st, act)
  D2C_WIDE(5); D2C_WIDE(6); D2C_WIDE(7); D2C_WIDE(8);
#undef D2C_WIDE
  return hipErrorInvalidValue;
}

// ---- few rows and a short contraction in float: one 16 x 16 tile per wave, every load of its contraction (at most kTileChunks
// chunks) requested at once.  Such a projection (37 rows x 768 x 256: 0.9 MB) is one memory latency long; gemm_rows_kernel, made
// to stream, spent several on its double-buffered chunks and ran on 8 to 24 compute units.  The activation rows (and row-major
// weights) come in whole rows and turn into operands in LDS, pre-tiled weights straight into registers.  Four neighbouring
// waves (64 columns) make a workgroup; the grid has one row of workgroups per 16 rows.  37 rows, pre-tiled: 768 x 256
// 9.8 -> 3.8 us, 1376 x 256 with the gate 9.8 -> 4.2, 256 x 256 7.1 -> 3.7, 256 x 688 6.9 -> 3.7 (activations in operand order:
// 5.7 to 6.6).
constexpr int kTileChunks = 4;
// More workgroups than this gain nothing over gemm_rows_kernel, which reads the weights once for all rows (37 rows x 4096 x 512
// in 384 workgroups 12.8 us, 10.0 there; 100 rows x 1376 x 256 in 154 7.5, 13.5 there).  Whole layers (pre-tiled) of 64 to 2048
// columns, FFN 80 to 2816, 1-128 rows, with this rule against without: 1.0 to 2.5 times as fast, none slower (768 columns, 17 rows 62 ->
// 56 us, 1024 columns, 16 rows 53 -> 49).  Row-major, 223 sizes of 1-128 rows x 64-4096 columns x 64-2048: 1.5 to 4 times, 2.4 on average.
constexpr int kTileWgs = 192;
// NORM, ROPE (one split, pre-tiled): the launches around such a projection are as long as it is, and a workgroup holds whole rows of
// its activations and, with heads of 64 columns and less, whole heads.  NORM: the activations are made here, every workgroup of a
// row tile for itself (16 rows, a few KB), and the first one leaves the updated residual rows in another buffer than the one that
// the others read.  ROPE: the output goes through LDS, and q, K and V rows leave turned, as launch_qkv_rope_scatter writes them.
// 37 rows of the small model, launches and the gaps between them apart: norm + QKV + RoPE 3.1 + 3.8 + 3.6 us -> 6.6, norm +
// gate/up 3.4 + 4.1 -> 7.3; two layers with 22 launches 91 us a call, 76 with 17.  Layers of 64 to 256 columns with 4 to 32 heads of
// 64, FFN 80 to 2816, 1-128 rows, the QKV projection so against three launches (graph): 4 to 21 % of the layer, none slower; the norm
// alone by the rule of norm_fuses.
struct RopeArgs {
  RopeSeqs seqs;
  const float *bias, *cos, *sin;
  int dq, dkv, head_dim;
  float* q_out;
};
template <int NC, int MODE, bool NORM, bool ROPE>
__global__ __launch_bounds__(256) void gemm_tile_kernel(const float* __restrict__ A, int lda, const float* __restrict__ W, int ldw,
                                                        float* __restrict__ P, int ldp, size_t split_stride, int m, int N, int K,
                                                        int k_per_split, float* __restrict__ act, const NormFuse norm,
                                                        const RopeArgs rope) {
  static_assert(MODE != kRowMajor || !(NORM || ROPE), "fused with pre-tiled weights only");
  constexpr int E = 4, KS = 16, KC = 64;
  constexpr int kPieces = NC * 16;                                  // 16-byte pieces of a row
  constexpr int kPitch = kPieces + 1;                               // in LDS: neighbouring rows on other banks
  __shared__ u32x4 a_lds[16 * kPitch];
  __shared__ u32x4 w_lds[MODE == kRowMajor ? 64 * kPitch : 1];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int n_base = (blockIdx.x * 4 + wave) * 16, row0 = blockIdx.y * 16;
  const int k_begin = blockIdx.z * k_per_split, k_end = min(K, k_begin + k_per_split);
  // nothing is read past the end of the contraction or of the rows (the last piece again, not used)
  Frag<float> b[NC * kSteps];
  u32x4 w_reg[MODE == kRowMajor ? NC * 4 : 1], a_reg[NC];
  if constexpr (MODE == kRowMajor) {
#pragma unroll
    for (int i = 0; i < NC * 4; ++i) {
      const int row = (i * 64 + lane) / kPieces, k = k_begin + (i * 64 + lane) % kPieces * E;
      w_reg[i] = ld16(W + (size_t)min(n_base + row, N - 1) * ldw + min(k, K - E));
    }
  } else {
    // chunks past the end of a short split lie past the end of the buffer and read as zeros: the activations are zeros there
    // too, and an infinite weight (of the last chunk, read again) times zero would be NaN
    const float* wtile = W + ((size_t)min(n_base / 16, (N + 15) / 16 - 1) * ldw + k_begin / KC) * (16 * KC);
    const int bytes = (k_end - k_begin + KC - 1) / KC * (16 * KC * 4);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wtile), 0, bytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < NC * kSteps; ++i)
      b[i].raw = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, lane * 16 + i * 1024, 0, 0));
  }
  // what the output's rows need: the chain of position and angles is over by the time the product is
  constexpr int kTurn = ROPE ? 2 : 1;                    // pairs of a thread: two of the 32 of a row's 64 columns
  const int t_row = threadIdx.x >> 4;
  int t_pos = 0, t_c1[kTurn] = {}, t_half = 0;
  float t_cos[kTurn], t_sin[kTurn];
  float *k_row = nullptr, *v_row = nullptr;
  if constexpr (ROPE) {
    const int row = min(row0 + t_row, m - 1), sq = rope_seq_of(rope.seqs, row);
    t_pos = rope.seqs.idx[sq][row - rope.seqs.off[sq]];
    k_row = static_cast<float*>(rope.seqs.k_cache[sq]) + (size_t)t_pos * rope.dkv;
    v_row = static_cast<float*>(rope.seqs.v_cache[sq]) + (size_t)t_pos * rope.dkv;
    t_half = rope.head_dim >> 1;
  }
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int at = i * 256 + (int)threadIdx.x, k = k_begin + at % kPieces * E;
    a_reg[i] = ld16((NORM ? norm.h + (size_t)min(row0 + at / kPieces, m - 1) * K : A + (size_t)min(row0 + at / kPieces, m - 1) * lda) +
                    min(k, K - E));
  }
  if constexpr (ROPE) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int pair = (threadIdx.x & 15) * 2 + e, head = pair / t_half, i = pair - head * t_half;
      t_c1[e] = head * rope.head_dim + i;                // column of the block; its pair's other one is t_half further on
      t_cos[e] = rope.cos[(size_t)t_pos * t_half + i];
      t_sin[e] = rope.sin[(size_t)t_pos * t_half + i];
    }
  }
  if constexpr (NORM) {
    if (norm.n_splits > 0) {
      f32x4 add[NC];
#pragma unroll
      for (int i = 0; i < NC; ++i) add[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int s = 0; s < norm.n_splits; ++s)
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int at = i * 256 + (int)threadIdx.x;
          add[i] += __builtin_bit_cast(f32x4, ld16(norm.P + s * norm.split_stride + (size_t)min(row0 + at / kPieces, m - 1) * norm.ldp +
                                                   min(at % kPieces * E, K - E)));
        }
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int at = i * 256 + (int)threadIdx.x, k = at % kPieces * E, row = row0 + at / kPieces;
        const f32x4 v = __builtin_bit_cast(f32x4, a_reg[i]) + add[i];
        if (norm.h_out != nullptr && blockIdx.x == 0 && row < m && k < K) *reinterpret_cast<f32x4*>(norm.h_out + (size_t)row * K + k) = v;
        a_reg[i] = __builtin_bit_cast(u32x4, v);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NC; ++i)
    if (k_begin + (i * 256 + (int)threadIdx.x) % kPieces * E >= k_end) a_reg[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int at = i * 256 + (int)threadIdx.x;
    a_lds[at / kPieces * kPitch + at % kPieces] = a_reg[i];
  }
  if constexpr (MODE == kRowMajor) {
#pragma unroll
    for (int i = 0; i < NC * 4; ++i) {
      const int row = (i * 64 + lane) / kPieces, piece = (i * 64 + lane) % kPieces;
      const u32x4 zero = {0u, 0u, 0u, 0u};
      w_lds[(wave * 16 + row) * kPitch + piece] = k_begin + piece * E < k_end ? w_reg[i] : zero;
    }
  }
  Frag<float> gain[NORM ? NC * kSteps : 1];
  if constexpr (NORM) {
#pragma unroll
    for (int i = 0; i < NC * kSteps; ++i) gain[i].raw = ld16(norm.gain + min((i * 4 + g) * E, K - E));
  }
  __syncthreads();
  __shared__ float inv_s[NORM ? 16 : 1];
  if constexpr (NORM) {
    // 16 threads a row; the zeros behind the row's end add nothing
    const int row = threadIdx.x >> 4, sub = threadIdx.x & 15;
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const f32x4 v = __builtin_bit_cast(f32x4, a_lds[row * kPitch + i * 16 + sub]);
      ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) ss += __shfl_xor(ss, o, kWave);
    if (sub == 0) inv_s[row] = 1.0f / sqrtf(ss / (float)K + norm.eps);
    __syncthreads();
  }
  Frag<float> a[NC * kSteps];
#pragma unroll
  for (int i = 0; i < NC * kSteps; ++i) {
    a[i].raw = a_lds[r * kPitch + i * 4 + g];
    if constexpr (NORM) {
      const f32x4 v = __builtin_bit_cast(f32x4, a[i].raw) * inv_s[r] * __builtin_bit_cast(f32x4, gain[i].raw);
      a[i].raw = (i * 4 + g) * E < K ? __builtin_bit_cast(u32x4, v) : u32x4{0u, 0u, 0u, 0u};
    }
    if (MODE == kRowMajor) b[i].raw = w_lds[(wave * 16 + r) * kPitch + i * 4 + g];
  }
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int i = 0; i < NC * kSteps; ++i) mfma16(acc[i & 1], a[i], b[i]);
  const f32x4 sum = acc[0] + acc[1];
  if constexpr (MODE == kPreSwiglu) {
    // column tiles alternate gate, up, gate, up ..: the odd wave of a pair hands the up values over
    __shared__ f32x4 xch[2][64];
    if (wave & 1) xch[wave >> 1][lane] = sum;
    __syncthreads();
    const int F = N >> 1, col = (n_base >> 5) * 16 + r;
    if ((wave & 1) || col >= F) return;
    const f32x4 u = xch[wave >> 1][lane];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = row0 + g * 4 + j;
      if (row < m) act[(size_t)row * F + col] = sum[j] / (1.0f + expf(-sum[j])) * u[j];
    }
    return;
  }
  if constexpr (ROPE) {
    __shared__ float turn[16][64 + 4];
#pragma unroll
    for (int j = 0; j < 4; ++j) turn[g * 4 + j][wave * 16 + r] = sum[j];
    __syncthreads();
    const int row = row0 + t_row;
    if (row >= m) return;
    float* const q_row = rope.q_out + (size_t)row * rope.dq;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int c1 = t_c1[e], n1 = blockIdx.x * 64 + c1;
      if (n1 >= N) continue;
      float x1 = 0.f, x2 = 0.f;
      if (rope.bias) {
        x1 = rope.bias[n1];
        x2 = rope.bias[n1 + t_half];
      }
      x1 += turn[t_row][c1];
      x2 += turn[t_row][c1 + t_half];
      const bool value = n1 >= rope.dq + rope.dkv;        // value rows are not turned
      const float o1 = value ? x1 : x1 * t_cos[e] - x2 * t_sin[e], o2 = value ? x2 : x2 * t_cos[e] + x1 * t_sin[e];
      float* const dst = n1 < rope.dq ? q_row + n1 : value ? v_row + (n1 - rope.dq - rope.dkv) : k_row + (n1 - rope.dq);
      dst[0] = o1;
      dst[t_half] = o2;
    }
    return;
  }
  const int col = n_base + r;
  if (col >= N) return;
  float* out = P + (size_t)blockIdx.z * split_stride;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = row0 + g * 4 + j;
    if (row < m) out[(size_t)row * ldp + col] = sum[j];
  }
}

template <int MODE, bool NORM = false, bool ROPE = false>
hipError_t launch_tile(const GemmPlan& pl, const void* A, int lda, const void* W, int ldw, float* P, int ldp, size_t split_stride, int m,
                       int N, int K, hipStream_t st, void* act, const NormFuse& norm = NormFuse{}, const RopeArgs& rope = RopeArgs{}) {
  const dim3 grid((N + 63) / 64, pl.row_chunks, pl.splits);
#define D2C_TILE(nc_)                                                                                                           \
  if (pl.k_per_split <= nc_ * 64) {                                                                                             \
    hipLaunchKernelGGL((gemm_tile_kernel<nc_, MODE, NORM, ROPE>), grid, dim3(256), 0, st, (const float*)A, lda, (const float*)W,  \
                       ldw, P, ldp, split_stride, m, N, K, pl.k_per_split, (float*)act, norm, rope);                            \
    return hipGetLastError();                                                                                                   \
  }
  D2C_TILE(1) D2C_TILE(2) D2C_TILE(3) D2C_TILE(4)
#undef D2C_TILE
  return hipErrorInvalidValue;
}

template <typename T, int MT, int NT, int WAVES, int MODE>
hipError_t launch_t(const GemmPlan& pl, const void* A, int lda, const void* W, int ldw, float* P, int ldp,
                    size_t split_stride, int m, int N, int K, hipStream_t st, void* act) {
  const int cols = 16 * NT * WAVES;
  const int n_blocks = (N + cols - 1) / cols;
  const int groups = (n_blocks * pl.splits + 7) / 8;            // weight tiles are dealt to the XCDs in groups of 8
  dim3 grid(groups * 8 * pl.row_chunks);
  if (NT >= 4)
    grid.x = 8 * ((groups + kSuperCols - 1) / kSuperCols) * ((pl.row_chunks + kSuperRows - 1) / kSuperRows) *
             (kSuperRows * kSuperCols);
  if constexpr (MODE == kRowStaged && kStageSlots<MT, NT, WAVES> == 0)
    return launch_t<T, MT, NT, WAVES, kRowMajor>(pl, A, lda, W, ldw, P, ldp, split_stride, m, N, K, st, act);
  else
  hipLaunchKernelGGL((gemm_rows_kernel<T, MT, NT, WAVES, MODE>), grid, dim3(WAVES * 64), 0, st, (const T*)A, lda,
                     (const T*)W, ldw, P, ldp, split_stride, m, N, K, pl.k_per_split, n_blocks, pl.splits,
                     pl.row_chunks, pl.rot, (T*)act);
  return hipGetLastError();
}

template <typename T, int NT, int WAVES, int MODE>
hipError_t launch_mt(const GemmPlan& pl, const void* A, int lda, const void* W, int ldw, float* P, int ldp,
                     size_t ss, int m, int N, int K, hipStream_t st, void* act) {
  switch (pl.mt) {
    case 1: return launch_t<T, 1, NT, WAVES, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    case 2: return launch_t<T, 2, NT, WAVES, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    case 3: return launch_t<T, 3, NT, WAVES, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    case 4: return launch_t<T, 4, NT, WAVES, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    case 5: return launch_t<T, 5, NT, WAVES, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    case 6: return launch_t<T, 6, NT, WAVES, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    case 7: return launch_t<T, 7, NT, WAVES, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    case 8: return launch_t<T, 8, NT, WAVES, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    default: break;
  }
  // 129-192 rows in one row chunk (bf16, one column tile per wave, 8 waves): even tile counts only
  if constexpr (sizeof(T) == 2 && NT == 1 && WAVES == 8) {
    switch (pl.mt) {
      case 10: return launch_t<T, 10, NT, WAVES, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
      case 12: return launch_t<T, 12, NT, WAVES, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <typename T, int MODE>
hipError_t launch_nt(const GemmPlan& pl, const void* A, int lda, const void* W, int ldw, float* P, int ldp,
                     size_t ss, int m, int N, int K, hipStream_t st, void* act) {
  if (pl.tile) {
    if constexpr (sizeof(T) == 4) return launch_tile<MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    return hipErrorInvalidValue;
  }
  if (pl.nt == 1) {
    if (pl.waves == 8) return launch_mt<T, 1, 8, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    if (pl.waves == 6) return launch_mt<T, 1, 6, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    if (pl.waves == 10) return launch_mt<T, 1, 10, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    if (pl.waves == 7) {
      if constexpr (MODE != kPreSwiglu) return launch_mt<T, 1, 7, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
      return hipErrorInvalidValue;
    }
    return launch_mt<T, 1, 4, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
  }
  if (pl.wide) {
    if constexpr (sizeof(T) == 2) {
      if (K % 128 || pl.k_per_split % 128) return hipErrorInvalidValue;
      // the staging wants whole 16-byte pieces and 32-bit offsets: other callers' buffers go through registers
      if ((uintptr_t)A % 16 == 0 && (size_t)m * lda * 2 < (1ull << 32))
        return launch_wide<MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
      GemmPlan other = pl;
      other.wide = false;
      if (K % 256 == 0 && pl.k_per_split % 256 == 0) {
        other.nt = 4;
        other.waves = 4;
        other.mt = std::max(6, pl.mt);
      } else {
        other.nt = 2;
        other.waves = 8;
        other.mt = 8;
      }
      other.row_chunks = (m + 16 * other.mt - 1) / (16 * other.mt);
      return launch_nt<T, MODE>(other, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
    }
    return hipErrorInvalidValue;
  }
  if (pl.nt == 4) {
    // 128 rows x 64 columns per wave, one wave per SIMD: only for full row chunks in bf16
    if constexpr (sizeof(T) == 2) {
      if (pl.waves == 4 && K % 256 == 0 && pl.k_per_split % 256 == 0) {
        if (pl.mt == 8) return launch_t<T, 8, 4, 4, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
        if (pl.mt == 7) return launch_t<T, 7, 4, 4, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
        if (pl.mt == 6) return launch_t<T, 6, 4, 4, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
      }
    }
    return hipErrorInvalidValue;
  }
  if (pl.waves == 8) return launch_mt<T, 2, 8, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
  return launch_mt<T, 2, 4, MODE>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, act);
}

template <typename T>
hipError_t launch_rows_staged(const GemmPlan& pl, const void* A, int lda, const void* W, int ldw, float* P, int ldp, size_t ss,
                              int m, int N, int K, hipStream_t st) {
  switch (pl.waves) {
    case 6: return launch_mt<T, 1, 6, kRowStaged>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, nullptr);
    case 7: return launch_mt<T, 1, 7, kRowStaged>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, nullptr);
    case 8: return launch_mt<T, 1, 8, kRowStaged>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, nullptr);
    case 10: return launch_mt<T, 1, 10, kRowStaged>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, nullptr);
    default: return launch_mt<T, 1, 4, kRowStaged>(pl, A, lda, W, ldw, P, ldp, ss, m, N, K, st, nullptr);
  }
}

// One 16-byte fragment per thread: dst block (tile t, chunk c) slot (step s, lane) <- src row
// row_of(t) + lane%16, bytes c*256 + s*64 + (lane/16)*16; rows >= N and bytes >= the row length read as zero.
// half > 0 (gate/up interleave, half % 16 == 0): dst tile 2j is src tile j, dst tile 2j+1 is the tile
// that starts at src row half + 16j.
__global__ __launch_bounds__(256) void preshuffle_kernel(const unsigned char* __restrict__ src, size_t src_pitch_bytes,
                                                         int N, size_t row_bytes, int chunks, int half,
                                                         unsigned char* __restrict__ dst, size_t n_frags) {
  const size_t f = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (f >= n_frags) return;
  const int lane = (int)(f & 63), s = (int)((f >> 6) & 3);
  const size_t block = f >> 8;
  const int c = (int)(block % chunks);
  const size_t t = block / chunks;
  const size_t row0 = half > 0 ? (t >> 1) * 16 + ((t & 1) ? (size_t)half : 0) : t * 16;
  const size_t row = row0 + (lane & 15);
  const size_t byte = (size_t)c * 256 + s * 64 + (lane >> 4) * 16;
  u32x4 v = {0u, 0u, 0u, 0u};
  if (row < (size_t)N && byte + 16 <= row_bytes) v = ld16(src + row * src_pitch_bytes + byte);
  *reinterpret_cast<u32x4*>(dst + f * 16) = v;
}

}  // namespace

// Row-major weights through LDS or in operand order.  The slots leave room for one workgroup on a compute unit where two fit
// without them, and a workgroup of few chunks is over before its queue is full, so short contractions lose: with 64-128
// elements of k on 1-128 rows x 65536 columns up to 11 %, a handful of workgroups (N = 64, 256) up to 20 % of 4 us; 7 row
// tiles (157 KB of LDS) still 11 % with 512.  From two chunks in one round of workgroups, or four in several, they gain (1-128
// rows x 4096 x 2048 10 %).  In float they gain with 5 row tiles and more in one round (5 %; 4-16 % lost in several), with fewer
// only where the round is full and not too long (6 %; 15 % lost on 1 and 17 rows x 16384 x 4096, 32 chunks each).
static bool staging_pays(int dtype, const GemmPlan& pl, int N) {
  const int wgs = ((N + 16 * pl.waves - 1) / (16 * pl.waves)) * pl.splits;
  const int chunks = pl.k_per_split / (dtype == kBF16 ? 128 : 64);
  if (dtype != kBF16) return wgs <= 256 && (pl.mt >= 5 || (wgs >= 200 && chunks >= 3 && chunks <= 16));
  if (wgs > 256) return chunks >= (pl.mt == 7 ? 8 : 4);
  return chunks >= 3 || (chunks == 2 && wgs >= 64);
}

// Chunks of k between the starts of neighbouring workgroups on row-major weights whose rows begin a power of two of 4 KB and
// more apart: workgroups that walk such rows in step ask for the same few memory channels.  Measured on 1-600 rows x 1024-126464
// columns, pitches of 4 to 64 KB, weights from memory, 976 sizes: geometric mean 1.04 over no moved starts, none below 0.98:
//   17 rows x 126464 x 4096 211 -> 178 us, 12288 x 4096 25 -> 21, 65536 x 8192 252 -> 167, 65536 x 2048 65 -> 52; 64 rows gain
//   10-45 % where 17 do, 100 rows 1-13 %, 256 x 126464 x 4096 412 -> 349, 512 x 126464 x 4096 685 -> 640; nothing at other
//   pitches (152064 x 3584, 4096 x 12288, 30000 x 1024).
// One apart does it, except at 4 KB (17 rows x 65536 x 2048: three 52 us, one 58).  Three apart meet again at 16 KB where a
// workgroup has 96 columns (17 rows x 24576 x 8192: none 79 us, one 68, three 82; 12288 x 8192 44, 37, 49).
// Where it loses: fewer than 16 chunks per workgroup are over before they fall into step (1 row x 8192 x 4096 in 8 chunks 17.0 ->
// 18.3 us); activations that fill an XCD's L2 (4 MB) stay there only while all workgroups read the same part of them (64 rows x 16384 x
// 32768 164 -> 228).  From 129 rows on the matrix cores weigh more: gains only on the widest matrices and, up to 192 rows, splits of
// 16 and 32 KB rows (150 x 12288 x 16384 152 -> 138), losses elsewhere (150 x 49152 x 4096 in two splits 131 -> 137, 200 x 4096 x
// 8192 1-2 %, 512 x 12288 x 32768 4 %, 1024 x 8192 x 4096 6 %).
static int start_chunks(const GemmPlan& pl, int dtype, int m, int N, int K) {
  const size_t pitch = (size_t)K * dtype_size(dtype);
  if (pitch < 4096 || (pitch & (pitch - 1)) != 0) return 0;
  const int chunks = pl.k_per_split / (dtype == kBF16 ? 128 : 64);
  bool pays;
  if (pl.row_chunks > 1)
    pays = pl.wide && pl.splits == 1 && (pl.row_chunks == 2 || (pl.row_chunks <= 4 && chunks >= 32 && pitch <= 32768));
  else if (pl.mt > 8)
    pays = chunks >= 16 && pitch <= 32768 && (pl.splits > 1 ? pitch >= 16384 : N >= 49152);
  else
    pays = chunks >= 16 && m * pitch < ((size_t)4 << 20);
  return !pays ? 0 : pitch == 4096 ? 3 : 1;
}

GemmPlan plan_gemm(const Tunables& t, int dtype, int m, int N, int K, bool single_split, bool row_major) {
  GemmPlan pl;
  const int tiles = (m + 15) / 16;
  pl.mt = tiles <= 8 ? (tiles < 1 ? 1 : tiles) : 8;
  pl.row_chunks = tiles <= 8 ? 1 : (tiles + 7) / 8;
  // 129-192 rows in bf16: still one row chunk (10 or 12 row tiles).  Two row chunks pull every weight tile through the L1 of two
  // compute units (us per layer at the LLaDA shape, one chunk and two: 144 rows 154 and 163, 160 rows 159 and 163; the Dream shape's
  // 37888 x 3584 and 3584 x 18944 together, 144 rows 146 and 156).  The line at 12 tiles dates from before the fragments were read
  // ahead; with that two chunks are the faster from 161 rows on (176 rows 172 and 168, 192 rows 177 and 169, Dream 176 rows 168 and
  // 159).  It still stands because it and the cost of a split below, too low from 129 rows on, decide this range together.
  if (tiles > 8 && tiles <= 12 && dtype == kBF16 && t.gemm_tall_chunk && (t.gemm_waves == 0 || t.gemm_waves == 8)) {
    pl.mt = tiles + (tiles & 1);
    pl.row_chunks = 1;
  }
  // two column tiles per wave halve the LDS reads per matrix-core step: a gain once there are several
  // row chunks (the kernel is LDS- and L2-bound there), a loss for a handful of rows (fewer waves in flight)
  pl.nt = (N > t.gemm_nt_big_n || pl.row_chunks > 1) ? 2 : 1;
  // several row chunks in bf16: 128 x 64 outputs per wave (gemm_wide_kernel or the rows kernel with four column tiles, see
  // below).  The latter takes chunks of k in pairs, the former any number of whole ones, measured on pairs as well.
  // Small row-major matrices are faster with two column tiles (512 rows x 1024 x 1024: 18 us, 22 and 25; 256 x 256 11, 13, 14).
  const bool wide = pl.row_chunks > 1 && m >= t.gemm_wide_min_rows && dtype == kBF16 && t.gemm_wide_tiles != 0 &&
                    K % 256 == 0 && !(row_major && t.gemm_wide_tiles == 1 && (size_t)N * K <= ((size_t)1 << 20));
  pl.wide = pl.tile = false;
  pl.rot = 0;
  // 8 waves share one activation chunk in LDS: fewer, fatter workgroups (about 1.5 per compute unit) with
  // fewer k splits measured faster than 4-wave groups at every projection shape of the two models
  // (7 waves only where no gated epilogue can follow: it pairs neighbouring waves)
  pl.waves = wide ? 8
             : (t.gemm_waves == 4 || t.gemm_waves == 6 || t.gemm_waves == 10 || (t.gemm_waves == 7 && !single_split))
                 ? t.gemm_waves
                 : 8;
  const int kc = dtype == kBF16 ? 128 : 64;                       // elements per 256-byte chunk
  const int chunks = (K + kc - 1) / kc;
  const int max_splits = single_split ? 1 : t.gemm_max_splits;
  // Up to 128 rows in float whose contraction, or a split of it, gemm_tile_kernel holds in flight at once.  Row-major weights
  // in several splits need the sum as a launch of its own and gain only where the other kernel reads them for many rows
  // (256 x 688: up to 64 rows 9.5 us there, 10.4 here; 100 rows 13.3 and 10.6).
  if (dtype != kBF16 && tiles <= 8 && t.gemm_waves == 0) {
    const int s = (chunks + kTileChunks - 1) / kTileChunks, cps = (chunks + s - 1) / s;
    if (s <= max_splits && (N + 63) / 64 * tiles * s <= kTileWgs && (!row_major || s == 1 || tiles > 4)) {
      pl.tile = true;
      pl.mt = pl.nt = 1;
      pl.waves = 4;
      pl.row_chunks = tiles;
      pl.k_per_split = cps * kc;
      pl.splits = (K + pl.k_per_split - 1) / pl.k_per_split;
      return pl;
    }
  }
  auto blocks_of = [&](int waves) { return (N + 16 * pl.nt * waves - 1) / (16 * pl.nt * waves); };
  auto splits_for = [&](int waves) {
    int s = 1;
    while (s < max_splits && blocks_of(waves) * (waves / 4) * pl.row_chunks * s < t.gemm_target_wgs && chunks / (s * 2) >= 2)
      s *= 2;
    return s;
  };
  int splits = splits_for(pl.waves);
  // Few rows (one row chunk, one column tile per wave): the kernel streams fastest when every compute unit
  // holds one workgroup of equal size, so the waves per workgroup and the split count are chosen together.
  // Cost of a shape = rounds of workgroups over the 256 units x (waves x chunks per split), +4 % per
  // additional split (its partial is written and read again; 4 % is too little from 129 rows on: 140 x 12288 x 4096 in 8 splits
  // 43.6 us, 128 rows in 2 28.5).  Measured at 48-69 rows: LLaDA QKV 25.1 ->
  // 22.5 us (6 waves x 2 splits = 256 workgroups instead of 8 x 2 = 192), Dream gate/up 68.6 -> 51.5 us
  // (10 waves = 237 workgroups in one round instead of 296 in two); 4-wave workgroups were slower at every
  // shape and are not searched.
  constexpr int kUnits = 256;
  if (pl.nt == 1 && pl.row_chunks == 1) {
    double best = 1e30;
    for (int w : {8, 6, 10, 7}) {                                 // 8 first: ties keep the 8-wave shape
      if (t.gemm_waves != 0 && w != pl.waves) continue;
      if (w == 7 && single_split) continue;
      if (pl.mt > 8 && w != 8) continue;                          // the tall chunk fits the registers of 8 waves only
      for (int s = 1; s <= max_splits; s *= 2) {
        const int cps = (chunks + s - 1) / s;
        if (s > 1 && cps < 2) break;
        const int eff = (chunks + cps - 1) / cps;
        const int wgs = blocks_of(w) * eff;
        const int rounds = (wgs + kUnits - 1) / kUnits;
        const double cost = (double)rounds * w * cps * (1.0 + 0.04 * (eff - 1));
        if (cost < best * 0.999) {
          best = cost;
          pl.waves = w;
          splits = s;
        }
      }
    }
  }
  // row tiles per row chunk when the tiles of m rows are dealt evenly to the chunks of so many workgroup rows
  auto dealt = [&](int pairs) { return std::max(5, (tiles + 2 * pairs - 1) / (2 * pairs)); };
  if (wide) {
    // Row chunks of 8 tiles, or of 7 or 6 where that makes their count a multiple of 8, the rows of the block of workgroups
    // that shares an XCD's L2, or keeps it.  Measured on the rows kernel at the LLaDA widths, 288-2048 rows: fewer tiles in
    // the same number of row chunks are a gain (288 rows as 3 x 6 tiles -14 %), more row chunks only up to a multiple of 8
    // (700 rows as 8 x 6 tiles instead of 6 x 8: -16 %; every other count lost 10-40 %).
    const int rc8 = (tiles + 7) / 8;
    int c = 8;
    if (rc8 % kSuperRows != 0)
      for (int x : {7, 6})
        if (c == 8 && ((tiles + x - 1) / x) % kSuperRows == 0) c = x;
    if (c == 8)
      for (int x : {6, 7})
        if (c == 8 && (tiles + x - 1) / x == rc8) c = x;

    // The rows kernel: splits by rounds of workgroups over the units, +7 % per additional split (the partials are as large
    // as the output and there are hundreds of rows of them).
    GemmPlan one = pl;
    one.mt = t.gemm_wide_mt != 0 ? t.gemm_wide_mt : c;
    one.row_chunks = (tiles + one.mt - 1) / one.mt;
    one.nt = one.waves = 4;
    one.splits = 1;
    double best = 1e30;
    for (int s = 1; s <= max_splits; s *= 2) {
      int cps = (chunks + s - 1) / s;
      cps += cps & 1;
      if (s > 1 && cps < 4) break;
      const int eff = (chunks + cps - 1) / cps;
      const int wgs = ((N + 255) / 256) * one.row_chunks * eff;
      const double cost = (double)((wgs + kUnits - 1) / kUnits) * cps * (1.0 + 0.07 * (eff - 1));
      if (cost < best * 0.999) {
        best = cost;
        one.splits = s;
      }
    }

    // gemm_wide_kernel: as many workgroup rows as pairs of those chunks, their tiles dealt evenly.  On this kernel the count is
    // not always the best: with pre-tiled weights of the LLaDA widths the best of 4 to 8 tiles is 6 % faster on average over
    // 257-2048 rows (777 rows x 4096 x 4096 43 us, 37 the best; 640 x 24576 x 4096 170, 129), with row-major ones 0 %.
    pl.wide = true;
    pl.mt = t.gemm_wide_mt != 0 ? t.gemm_wide_mt : dealt(((tiles + c - 1) / c + 1) / 2);
    pl.row_chunks = (tiles + pl.mt - 1) / pl.mt;
    // Columns per workgroup and splits by a time model in us, a workgroup taking two row chunks: a chunk of k costs a
    // row tile 0.35 us with 256 columns and 0.8 of that with 192 (measured, 512 rows: 105 us for gate/up as 192 workgroups
    // of 256 columns, 93 as 256 of 192: what counts is full rounds over the 256 units), and every split writes and
    // reads m x N partial sums at about 5.5 TB/s.  Any count of splits: Dream's QKV at 768 rows runs 3.
    const int pairs = (pl.row_chunks + 1) / 2;
    const double chunk_us = 0.35 * pl.mt, split_us = single_split ? 0.0 : (double)tiles * 16 * N * 8e-6 / 5.5;
    best = 1e30;
    for (int nt : {4, 3})
      for (int s = 1; s <= max_splits; ++s) {
        int cps = (chunks + s - 1) / s;
        cps += cps & 1;                                           // splits start on pairs of chunks
        if (s > 1 && cps < 4) break;
        const int eff = (chunks + cps - 1) / cps;
        const int wgs = ((N + 64 * nt - 1) / (64 * nt)) * pairs * eff;
        const double cost = (double)((wgs + kUnits - 1) / kUnits) * cps * chunk_us * (nt == 3 ? 0.8 : 1.0) + split_us * eff;
        if (cost < best * 0.999) {
          best = cost;
          splits = s;
          pl.nt = nt;
        }
      }

    // The line between the two: time in us, fitted to both kernels on 257-12288 rows and 100 matrices from 16 x 256 to
    // 37888 x 3584 (1926 sizes; 96 % of the predictions within 15 %).  A round of workgroups costs a start, per chunk of k a
    // part per row tile and one for the columns (row-major weights, read in operand order, make that the larger), and per row
    // tile the gate; a round that does not fill the chip costs `tail` and its share of the rest; a split costs a part and its
    // partial sums.  gemm_wide_kernel has half the workgroups, so it loses where these no longer fill the chip: 1024 rows x
    // 8192 x 4096 65 us in the rows kernel, 78 in the other, but 512 x 12288 x 4096 89 and 62.  Taking the cheaper by this
    // gains 23 % pre-tiled over the rows kernel alone, always the faster 23.5 %, gemm_wide_kernel alone 21 %; row-major 12, 13
    // and 7 %.  Its mistakes cost up to 8 % against the rows kernel (10 % row-major, in 12 sizes of the 1926 above 3 %).
    struct Cost { double start, round, tile, cols, gate, tail, split, part, out; };
    static constexpr Cost one_pre{1.6, 5.6, 0.195, 0.11, 0.25, 0.7, 4.5, 0.23, 0.10}, wide_pre{0.0, 5.1, 0.31, 0.20, 0.95, 0.7, 2.5, 0.28, 0.13},
        one_rows{2.2, 6.9, 0.106, 1.48, 0.0, 0.8, 4.5, 0.22, 0.10}, wide_rows{0.5, 7.0, 0.166, 2.92, 0.0, 0.8, 3.0, 0.26, 0.12};
    auto shape_us = [&](const GemmPlan& q, int s, const Cost& k) {
      int cps = (chunks + s - 1) / s;
      cps += cps & 1;
      const int eff = (chunks + cps - 1) / cps;
      const int rows = (q.row_chunks + q.chunks_per_wg() - 1) / q.chunks_per_wg(), cols = q.cols_per_wg();
      const int per_xcd = (((N + cols - 1) / cols) * eff + 7) / 8;      // weight tiles of an XCD
      // an XCD's workgroups go to its four groups of 8 units in turn: workgroups that leave at once (padding of the blocks of
      // kSuperRows rows) give the groups unequal shares
      const double full = !q.wide || rows > kSuperRows ? per_xcd * ((rows + 3) / 4) / 8.0 : per_xcd * rows / 32.0;
      const double whole = std::floor(full), rest = full - whole;
      const double rounds = whole < 1.0 ? 1.0 : whole + (rest > 0.0 ? k.tail + (1.0 - k.tail) * rest : 0.0);
      const double width = q.nt == 3 ? 0.8 : 1.0, mb = 4e-6 * (tiles * 16) * N;
      return k.start + rounds * (k.round + width * (cps * (k.tile * q.mt + k.cols) + (single_split ? k.gate * q.mt : 0.0))) +
             (eff > 1 ? k.split + k.part * mb * eff : 0.0) + k.out * mb * (single_split ? 0.25 : 1.0);
    };
    const double one_us = shape_us(one, one.splits, row_major ? one_rows : one_pre);
    const double wide_us = shape_us(pl, splits, row_major ? wide_rows : wide_pre) * (row_major ? 1.03 : 1.0);
    if (t.gemm_wide_tiles == 3 || (t.gemm_wide_tiles != 2 && one_us < wide_us)) {
      pl = one;
      splits = one.splits;
    }
  }
  int chunks_per_split = (chunks + splits - 1) / splits;
  if (wide) chunks_per_split += chunks_per_split & 1;
  pl.k_per_split = chunks_per_split * kc;
  pl.splits = (K + pl.k_per_split - 1) / pl.k_per_split;
  // Two row chunks (193-256 rows) are one workgroup of the wide kernel as well: where that fills the chip (the head on all
  // masked rows of a first step, 256 rows x 126464 columns: 374 -> 317 us), not for a block's matrices (96 column
  // blocks at most).
  if (!wide && dtype == kBF16 && pl.nt == 2 && pl.row_chunks == 2 && K % kc == 0 &&
      ((t.gemm_wide_tiles == 1 && ((N + 255) / 256) * pl.splits >= 3 * kUnits / 4) || t.gemm_wide_tiles == 2)) {
    pl.wide = true;
    pl.mt = dealt(1);
    pl.nt = 4;
    pl.waves = 8;
  }
  pl.rot = t.gemm_rot >= 0 ? t.gemm_rot : row_major ? start_chunks(pl, dtype, m, N, K) : 0;
  return pl;
}

hipError_t launch_gemm(int dtype, const GemmPlan& pl, const void* A, int lda, const void* W, int ldw, float* P,
                       int ldp, size_t split_stride, int m, int N, int K, hipStream_t st, bool pre) {
  if (m <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
  const int e = dtype == kBF16 ? 8 : 4;
  // 16-byte fragments: the contraction length and both pitches must be whole fragments
  if (K % e || lda % e || (!pre && ldw % e)) return hipErrorInvalidValue;
  if (pl.mt * 16 * pl.row_chunks < m || (size_t)pl.k_per_split * pl.splits < (size_t)K) return hipErrorInvalidValue;
  if (split_stride < (size_t)m * ldp || ldp < N) return hipErrorInvalidValue;
  if (pre) {
    // ldw = chunks per tile of the pre-tiled copy; every split must start on a chunk boundary
    const int kc = dtype == kBF16 ? 128 : 64;
    if (ldw != (K + kc - 1) / kc || pl.k_per_split % kc) return hipErrorInvalidValue;
    if (dtype == kBF16)
      return launch_nt<bf16, kPre>(pl, A, lda, W, ldw, P, ldp, split_stride, m, N, K, st, nullptr);
    return launch_nt<float, kPre>(pl, A, lda, W, ldw, P, ldp, split_stride, m, N, K, st, nullptr);
  }
  if (pl.nt == 1 && !pl.tile && (uintptr_t)W % 16 == 0 && (size_t)ldw * dtype_size(dtype) * 16 < (1ull << 31) &&
      staging_pays(dtype, pl, N)) {
    if (dtype == kBF16)
      return launch_rows_staged<bf16>(pl, A, lda, W, ldw, P, ldp, split_stride, m, N, K, st);
    return launch_rows_staged<float>(pl, A, lda, W, ldw, P, ldp, split_stride, m, N, K, st);
  }
  if (dtype == kBF16)
    return launch_nt<bf16, kRowMajor>(pl, A, lda, W, ldw, P, ldp, split_stride, m, N, K, st, nullptr);
  return launch_nt<float, kRowMajor>(pl, A, lda, W, ldw, P, ldp, split_stride, m, N, K, st, nullptr);
}

hipError_t launch_gemm_swiglu(int dtype, const GemmPlan& pl, const void* A, int lda, const void* W, int ldw,
                              void* act, int F, int m, int K, hipStream_t st) {
  if (m <= 0 || F <= 0 || K <= 0 || F % 16) return hipErrorInvalidValue;
  const int e = dtype == kBF16 ? 8 : 4, kc = dtype == kBF16 ? 128 : 64;
  if (K % e || lda % e || ldw != (K + kc - 1) / kc) return hipErrorInvalidValue;
  if (pl.splits != 1 || pl.mt * 16 * pl.row_chunks < m || pl.k_per_split < K)
    return hipErrorInvalidValue;
  if (dtype == kBF16)
    return launch_nt<bf16, kPreSwiglu>(pl, A, lda, W, ldw, nullptr, 0, 0, m, 2 * F, K, st, act);
  return launch_nt<float, kPreSwiglu>(pl, A, lda, W, ldw, nullptr, 0, 0, m, 2 * F, K, st, act);
}

bool gemm_fuses(int dtype, const GemmPlan& pl) { return dtype == kF32 && pl.tile && pl.splits == 1; }
// Every column block adds up the splits of its rows for itself.  Device us of a layer with the norm inside gate/up less without
// (1-128 rows, FFN 80-2816, launches from a graph; the launch itself costs the host about 2):
//   splits      1      2      4      8
//   K =  64   -1.2   -1.8   -1.7   -0.1
//   K = 128   -1.0   -1.0   -0.9   +1.2
//   K = 192   -0.5   -0.5   -0.3   +1.5
//   K = 256   +0.6   +1.3   +2.5   +7.4   (32 heads of 64: 36 rows 38 us without, 46 with)
// With 256 columns it is taken for the host's sake, and only where the fused QKV projection gives the device more (3-5 us a layer)
// than this takes: heads of 128, which are not fused, lost 2-5 % in a graph.
bool norm_fuses(int n_splits, int K, bool qkv_fused) { return n_splits <= (K <= 64 ? 8 : K <= 192 ? 4 : qkv_fused ? 2 : 0); }
bool rope_fuses(int head_dim, int n_calls) { return head_dim % 2 == 0 && 64 % head_dim == 0 && n_calls > 0 && n_calls <= kRopeMaxSeqs; }

hipError_t launch_gemm_tile_fused(const GemmPlan& pl, const NormFuse* norm, const float* A, int lda, const void* W, int ldw,
                                  const RopeFuse* rope, float* act, int m, int N, int K, hipStream_t st) {
  if (m <= 0 || N <= 0 || K <= 0 || K % 4 || !gemm_fuses(kF32, pl) || pl.row_chunks * 16 < m || pl.k_per_split < K ||
      ldw != (K + 63) / 64 || (norm ? norm->n_splits > 0 && norm->ldp < K : lda % 4 != 0 || lda < K) || !rope == !act ||
      (act && (!norm || N % 32)))
    return hipErrorInvalidValue;
  // h_out: others still read h, and without partial sums there is nothing to update
  if (norm && (norm->h_out == norm->h || (norm->h_out && norm->n_splits == 0) || (norm->ldp | norm->split_stride) % 4))
    return hipErrorInvalidValue;
  if (act) return launch_tile<kPreSwiglu, true, false>(pl, A, lda, W, ldw, nullptr, 0, 0, m, N, K, st, act, *norm);
  RopeArgs ra{};
  const int dq = rope->n_heads * rope->head_dim, dkv = rope->n_kv_heads * rope->head_dim;
  if (!rope_fuses(rope->head_dim, rope->n_calls) || !rope_seqs(rope->calls, rope->n_calls, ra.seqs) ||
      ra.seqs.off[rope->n_calls] != m || N != dq + 2 * dkv)
    return hipErrorInvalidValue;
  ra.bias = rope->bias; ra.cos = rope->rope_cos; ra.sin = rope->rope_sin;
  ra.dq = dq; ra.dkv = dkv; ra.head_dim = rope->head_dim; ra.q_out = rope->q_out;
  return norm ? launch_tile<kPre, true, true>(pl, A, lda, W, ldw, nullptr, 0, 0, m, N, K, st, nullptr, *norm, ra)
              : launch_tile<kPre, false, true>(pl, A, lda, W, ldw, nullptr, 0, 0, m, N, K, st, nullptr, NormFuse{}, ra);
}

size_t preshuffled_bytes(int N, int K, int dtype) {
  const size_t row_bytes = (size_t)K * dtype_size(dtype);
  return (size_t)((N + 15) / 16) * ((row_bytes + 255) / 256) * 4096;
}

hipError_t launch_preshuffle(int dtype, const void* W, int ldw, int N, int K, void* dst, hipStream_t st,
                             int interleave_half) {
  if (N <= 0 || K <= 0 || ldw < K) return hipErrorInvalidValue;
  if (interleave_half < 0 || interleave_half % 16 || (interleave_half && N != 2 * interleave_half))
    return hipErrorInvalidValue;
  const size_t ts = dtype_size(dtype);
  if ((size_t)K * ts % 16 || (size_t)ldw * ts % 16) return hipErrorInvalidValue;
  const size_t n_frags = preshuffled_bytes(N, K, dtype) / 16;
  const int chunks = (int)(((size_t)K * ts + 255) / 256);
  hipLaunchKernelGGL(preshuffle_kernel, dim3((unsigned)((n_frags + 255) / 256)), dim3(256), 0, st,
                     (const unsigned char*)W, (size_t)ldw * ts, N, (size_t)K * ts, chunks, interleave_half,
                     (unsigned char*)dst, n_frags);
  return hipGetLastError();
}

}  // namespace d2c
