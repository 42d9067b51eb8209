// Observation-window scoring on the matrix cores for bf16 at head size 64 and for fp32 (Eq. 1-2; Algorithm 1:
// softmax(Q_win K^T).mean(-2).pooling(-1)). The operation and the two sweeps over the keys are those of score_mfma.hip,
// which serves bf16 at head size 128.
//
// A wavefront holds its keys in registers, in matrix operand layout, and takes all rows of the Q block past them (Q in
// LDS): the keys come straight from global memory, without a detour through LDS and without barriers between tiles.
// fp32 operands are split into three bf16 terms each (8 + 8 + 8 bits of significand: the split is exact), and six of
// the nine products are taken, all but those below 2^-24 of the whole: per 16 elements six MFMAs of 32 cycles instead
// of the eight of 64 cycles that the fp32 form needs. Scores differ from float64 ones by 3.4e-7 (2-norm; 4.0e-7 with
// the fp32 multiply-adds of the vector ALU).
// The split, and sums of products in the matrix pipe's own order, end before the range of the elements does: what they
// leave without a number is taken again as fp32 multiply-adds (see logit_fma).
//
// Measured, both sweeps of a call, 128 rows, one MI355X: fp32, 8 layers of 8192 tokens, 8 heads of 128: 215 us (2270 us on
// the vector ALU, score_generic.hip); bf16, 16 layers of 16384 tokens, 8 heads of 64: 131 us = 4.1 TB/s (1690 us). Bound:
// fp32 by the matrix pipe (80 us of MFMAs), bf16 by the vector ALU's share of a unit (32 keys x 32 rows: 16 multiply-adds,
// exponentials and adds per lane).
//
//   stats kernel: S_tile = K_tile . Q^T  (keys as the MFMA M index, rows as N: a lane holds ONE row and 16
//                 keys, so the row maximum / sum of exponentials is an in-lane reduction); every workgroup writes
//                 one partial (max, sum) per row for its chunk of keys;
//   merge:        the chunk partials of a (sequence, head) become lse2[row] (kernel boundaries are the only
//                 synchronisation between workgroups): in the emit kernel for a single layer, in a small kernel of
//                 its own when a call covers several layers;
//   emit kernel:  S_tile = Q . K_tile^T (rows as M, keys as N: a lane holds ONE key and 16 rows, so the sum over
//                 the rows is an in-lane reduction), p = exp2(S * c - lse2[row]), window/group sum, max-pool,
//                 write.
#include "score_common.h"

#include <type_traits>

namespace dkv {

constexpr int kWaves = 8;             // wavefronts per workgroup
constexpr int kThreads = kWaves * 64;
constexpr int kTileRow = kWaves * 32; // keys of one tile of every wavefront: a chunk is a whole number of these
static_assert(kTileRow >= kMfmaMinChunk && kTileRow >= kGenericKeys, "the workspace is sized for chunks of so many keys");

// Q and K of the layers one launch covers (kernel argument, indexed by the layer's place in the launch).
struct TileLayers {
  const char* q[DKV_MAX_SELECT_LAYERS];
  const char* k[DKV_MAX_SELECT_LAYERS];
};

// ------------------------------------------------------------------------------------------------------
// Chunks and tasks. Every sequence is cut into chunks of `chunk` keys (all S of them, window included); a task is
// one chunk of one KV head in one layer. Linear order of tasks: layer slowest, then chunk (over all sequences), KV
// head fastest - with 8 KV heads a head's chunks then run on one XCD, whose L2 holds that head's Q.
// ------------------------------------------------------------------------------------------------------
// Lane l of every wavefront holds sequence s0 + l: the number of its first chunk, its first token, its length.
struct ChunkMap {
  int first, begin, len;
  int total;                                    // chunks of all sequences up to these
};

__device__ inline ChunkMap chunk_map(const int32_t* __restrict__ cu, int n_seqs, int s0, int base, int chunk) {
  const int s = s0 + (int)(threadIdx.x & 63);
  ChunkMap m;
  m.begin = s < n_seqs ? cu[s] : 0;
  m.len = s < n_seqs ? cu[s + 1] - m.begin : 0;
  const int n = (m.len + chunk - 1) / chunk;
  const int incl = wave_prefix_sum(n);
  m.first = s < n_seqs ? base + incl - n : 0x7fffffff;
  m.total = base + __builtin_amdgcn_readlane(incl, 63);
  return m;
}

__device__ inline int all_chunks(const int32_t* __restrict__ cu, int n_seqs, int chunk, const ChunkMap& m) {
  int total = m.total;
  for (int s0 = 64; s0 < n_seqs; s0 += 64) total = chunk_map(cu, n_seqs, s0, total, chunk).total;
  return total;
}

struct Task {
  int layer, seq, head;
  int chunk_id;          // over all sequences
  int c0, len;           // first key of the chunk within the sequence, keys of the chunk
  int begin, S;          // first token of the sequence, its length
};

__device__ inline Task find_task(const int32_t* __restrict__ cu, int n_seqs, int chunk, ChunkMap m, int n_chunks, int Hkv,
                                 int task) {
  Task t;
  const int per_layer = n_chunks * Hkv;
  t.layer = task / per_layer;
  const int r = task - t.layer * per_layer;
  t.chunk_id = r / Hkv;
  t.head = r - t.chunk_id * Hkv;
  int s0 = 0;
  while (t.chunk_id >= m.total) {               // batches of more than 64 sequences
    s0 += 64;
    m = chunk_map(cu, n_seqs, s0, m.total, chunk);
  }
  // the last sequence of the 64 that starts at or before the chunk (sequences without chunks share their start with
  // the next one; lanes past the batch start at infinity)
  const int lane = 63 - __builtin_clzll(__ballot(m.first <= t.chunk_id));
  t.seq = s0 + lane;
  t.begin = __builtin_amdgcn_readlane(m.begin, lane);
  t.S = __builtin_amdgcn_readlane(m.len, lane);
  t.c0 = (t.chunk_id - __builtin_amdgcn_readlane(m.first, lane)) * chunk;
  t.len = t.S - t.c0 < chunk ? t.S - t.c0 : chunk;
  return t;
}

// ------------------------------------------------------------------------------------------------------
// Operands
// ------------------------------------------------------------------------------------------------------
// Element types: bytes in memory, bf16 terms per element in the products.
struct ElemBf16 {
  static constexpr int kBytes = 2, kTerms = 1;
};
struct ElemF32 {
  static constexpr int kBytes = 4, kTerms = 3;
};

// NT: key tiles (of 32 keys) per wavefront and task. A stage is what a wavefront takes through the rows at once: kTiles
// tiles, so that a fragment of Q read from LDS serves both. bf16: two slots of registers hold a stage each; the loads of
// a slot start when its stage has been used up (kEnd of them) and go on during the stage of the other slot: kFirst next
// to the products of its first row tile, the rest next to the exponentials of its last one. All at once they would fill
// the queue of the compute unit, which takes about 64 KB: past that a load instruction blocks its wavefront until
// earlier ones have returned (measured: 8 wavefronts with 4 loads of 1 KB each issue them in 150 cycles, with 16 each in
// 9000), and nothing is computed meanwhile. fp32: one tile per stage and task; the split terms are a copy, so the slot
// is free for the next task's keys as soon as they are made.
template <typename E, int D, int NT>
struct Geo {
  static constexpr int kSteps = D / 16;                        // MFMA steps over the head dimension
  static constexpr int kTerms = E::kTerms;
  static constexpr int kTiles = kTerms == 1 && NT > 1 ? 2 : 1;
  static constexpr int kPerTask = NT / kTiles;                 // stages per task
  static constexpr int kSlots = kTerms == 1 ? 2 : 1;
  static constexpr int kChunk = NT * kTileRow;
  static constexpr int kStepBytes = 16 * E::kBytes;            // bytes of a key row per step
  static constexpr int kTileLoads = kSteps * E::kBytes / 2;    // 16-byte loads per tile and lane: one or two per step
  static constexpr int kLoads = kTiles * kTileLoads;
  static constexpr int kEnd = kSlots == 2 ? (3 * kLoads + 7) / 8 : 0, kFirst = (kLoads - kEnd + 1) / 2;
  static constexpr int kQRow = D * 2 + 16;                     // bytes per row and term of Q in LDS (16 of padding: conflict-free 16-byte reads)
  static constexpr int kQPieces = D * E::kBytes / 16;          // 16-byte pieces per row of Q in memory
  static constexpr int kMaxRows = kTerms * D > 256 ? 128 : 256;   // 8 pieces of Q a thread, as at head size 64 (in LDS three terms of 160 rows of 128 elements would fit)
  static constexpr int kQLoads = kMaxRows * kQPieces / kThreads;  // pieces per thread of the widest Q block
  static_assert(kPerTask <= 2 && (kTerms == 1 || NT == 1), "a task is one or two stages, and one of one tile for split elements");
};

// Keys of a stage as they are loaded: lane l holds, for step j, elements 16 j + 8 (l / 32) .. + 7 of key l % 32 of every
// tile. A wavefront-wide load touches 32 rows; the steps of a tile complete the rows' cache lines, and the stream runs
// as fast as one of fully coalesced rows (6.15 against 6.27 TB/s over 2.1 GB).
template <typename G>
struct Slot {
  uint4 v[G::kTiles][G::kTileLoads];
};

// What is still to be loaded into a slot: the rows of this lane.
template <typename G>
struct Pending {
  const char* base;
  uint32_t off[G::kTiles];
};

// Key (within the chunk) of lane 0's column of tile `tile` of wavefront `wave`.
__device__ inline int tile_key(int tile, int wave) { return tile * kTileRow + wave * 32; }

// The tiles of stage s of a chunk; keys past the chunk repeat its last one.
template <typename G>
__device__ inline void set_pending(Pending<G>& pend, const char* base, uint32_t stride_b, int s, int wave, int len) {
  pend.base = base;
#pragma unroll
  for (int i = 0; i < G::kTiles; ++i) {
    const int key = tile_key(s * G::kTiles + i, wave) + (int)(threadIdx.x & 31);
    pend.off[i] = (uint32_t)(key < len ? key : len - 1) * stride_b + (threadIdx.x & 32u) * G::kStepBytes / 64;
  }
}

// Loads [from, to) of a slot, in the order in which the products use them: step by step, all tiles.
template <typename G>
__device__ inline void load_some(Slot<G>& slot, const Pending<G>& pend, int from, int to) {
  constexpr int kPerStep = G::kTileLoads / G::kSteps;
#pragma unroll
  for (int i = 0; i < G::kLoads; ++i) {
    const int j = i / (G::kTiles * kPerStep), tile = i / kPerStep % G::kTiles, part = i % kPerStep;
    if (i >= from && i < to)
      slot.v[tile][j * kPerStep + part] =
          *reinterpret_cast<const uint4*>(pend.base + pend.off[tile] + (j * G::kStepBytes + part * 16));
  }
}

// x as three bf16 terms, two elements at a time: hi + mid + lo == x, from 2^-110 (below it the smallest bits of lo are
// lost) to where hi rounds to infinity (3.396e38).
__device__ inline uint32_t pack_bf16(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 v;
  v[0] = (__bf16)a;
  v[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, v);
}
__device__ inline void split_pair(uint32_t xa, uint32_t xb, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  float a = __uint_as_float(xa), b = __uint_as_float(xb);
  hi = pack_bf16(a, b);
  a -= __uint_as_float(hi << 16);
  b -= __uint_as_float(hi & 0xffff0000u);
  mid = pack_bf16(a, b);
  a -= __uint_as_float(mid << 16);
  b -= __uint_as_float(mid & 0xffff0000u);
  lo = pack_bf16(a, b);
}

// Keys of a stage as operands of the products.
template <typename G>
struct Keys {
  uint4 t[G::kTerms][G::kTiles][G::kSteps];
};

template <typename G>
__device__ inline void make_keys(const Slot<G>& slot, Keys<G>& k) {
#pragma unroll
  for (int i = 0; i < G::kTiles; ++i)
#pragma unroll
    for (int j = 0; j < G::kSteps; ++j) {
      if constexpr (G::kTerms == 1) {
        k.t[0][i][j] = slot.v[i][j];
      } else {
        const uint4 a = slot.v[i][2 * j], b = slot.v[i][2 * j + 1];
        split_pair(a.x, a.y, k.t[0][i][j].x, k.t[1][i][j].x, k.t[2][i][j].x);
        split_pair(a.z, a.w, k.t[0][i][j].y, k.t[1][i][j].y, k.t[2][i][j].y);
        split_pair(b.x, b.y, k.t[0][i][j].z, k.t[1][i][j].z, k.t[2][i][j].z);
        split_pair(b.z, b.w, k.t[0][i][j].w, k.t[1][i][j].w, k.t[2][i][j].w);
      }
    }
}

// The Q block of a task. Rows past the last one repeat it (what they give is never used: the statistics of such rows
// are not read, and the emit kernel gives them a normaliser of +inf). In LDS: [kTerms][row_tiles * 32][kQRow].
template <typename G>
struct QBlock {
  uint4 v[G::kQLoads];
};

template <typename G>
__device__ inline void load_q(QBlock<G>& q, const char* __restrict__ q_head, int rows, int row_tiles) {
  uint32_t tid = threadIdx.x;
  asm volatile("" : "+v"(tid));   // the addresses are rebuilt here: kept across the caller's loop they cost registers
#pragma unroll
  for (int i = 0; i < G::kQLoads; ++i) {
    q.v[i] = make_uint4(0, 0, 0, 0);
    if (i * kThreads < row_tiles * 32 * G::kQPieces) {                    // uniform
      const uint32_t pc = tid + i * kThreads;
      uint32_t row = pc / G::kQPieces;
      row = row < (uint32_t)rows ? row : rows - 1;
      q.v[i] = *reinterpret_cast<const uint4*>(q_head + (row * G::kQPieces + pc % G::kQPieces) * 16u);
    }
  }
}

template <typename G>
__device__ inline void store_q(const QBlock<G>& q, char* __restrict__ qbuf, int row_tiles) {
  uint32_t tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
#pragma unroll
  for (int i = 0; i < G::kQLoads; ++i) {
    const uint32_t pc = tid + i * kThreads;
    if (pc < (uint32_t)(row_tiles * 32 * G::kQPieces)) {
      char* dst = qbuf + (pc / G::kQPieces) * G::kQRow;
      if constexpr (G::kTerms == 1) {
        *reinterpret_cast<uint4*>(dst + (pc % G::kQPieces) * 16) = q.v[i];
      } else {
        uint2 hi, mid, lo;
        split_pair(q.v[i].x, q.v[i].y, hi.x, mid.x, lo.x);
        split_pair(q.v[i].z, q.v[i].w, hi.y, mid.y, lo.y);
        dst += (pc % G::kQPieces) * 8;
        *reinterpret_cast<uint2*>(dst) = hi;
        *reinterpret_cast<uint2*>(dst + row_tiles * 32 * G::kQRow) = mid;
        *reinterpret_cast<uint2*>(dst + 2 * row_tiles * 32 * G::kQRow) = lo;
      }
    }
  }
}

// Fragment j of a row tile of Q, all terms (qrow: this lane's row and half; plane: bytes from one term to the next).
template <typename G>
struct QFrag {
  uint4 t[G::kTerms];
};
template <typename G>
__device__ inline QFrag<G> q_frag(const char* __restrict__ qrow, int plane, int j) {
  QFrag<G> f;
#pragma unroll
  for (int i = 0; i < G::kTerms; ++i) f.t[i] = *reinterpret_cast<const uint4*>(qrow + i * plane + j * 32);
  return f;
}

// Step j of the products of one row tile of Q with the tiles of a stage. KEYS_AS_M: a lane holds one row and, in
// register i, key 8 (i / 4) + 4 (lane / 32) + i % 4; otherwise one key and rows in that order.
template <typename G, bool KEYS_AS_M>
__device__ inline void multiply_step(int j, const QFrag<G>& q, const Keys<G>& k, floatx16 (&acc)[G::kTiles]) {
#pragma unroll
  for (int p = 0; p < G::kTiles; ++p) {
    if (j == 0)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[p][i] = 0.0f;
    auto product = [&](int a, int b) {
      const bf16x8 qq = __builtin_bit_cast(bf16x8, q.t[a]), kk = __builtin_bit_cast(bf16x8, k.t[b][p][j]);
      acc[p] = KEYS_AS_M ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk, qq, acc[p], 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qq, kk, acc[p], 0, 0, 0);
    };
    if constexpr (G::kTerms == 3) {          // the smallest first
      product(0, 2);
      product(2, 0);
      product(1, 1);
      product(0, 1);
      product(1, 0);
    }
    product(0, 0);
  }
}

// All steps; beside(j) is issued next to step j.
template <typename G, bool KEYS_AS_M, typename Beside>
__device__ inline void multiply(const char* __restrict__ qrow, int plane, const Keys<G>& k, floatx16 (&acc)[G::kTiles], Beside beside) {
  constexpr int kAhead = G::kTerms == 1 ? 3 : 2;
  QFrag<G> q[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) q[i] = q_frag<G>(qrow, plane, i);
#pragma unroll
  for (int j = 0; j < G::kSteps; ++j) {
    multiply_step<G, KEYS_AS_M>(j, q[j % kAhead], k, acc);
    if (j + kAhead < G::kSteps) q[j % kAhead] = q_frag<G>(qrow, plane, j + kAhead);
    beside(j);
  }
}

// Row tile t + 1 into `y`, slice by slice, next to the work on row tile t: work(j) is the share of slice j. Matrix pipe
// and vector ALU are busy together within one wavefront: without the interleaving the two wavefronts of a SIMD take
// their products at the same time and their exponentials at the same time (half-wave units of 32 x 32 x 128: 560 cycles
// of a SIMD instead of 380).
template <typename G, bool KEYS_AS_M, bool MORE, typename Work, typename Loads>
__device__ inline void interleave(const char* __restrict__ qnext, int plane, const Keys<G>& k, floatx16 (&y)[G::kTiles], Work work,
                                  Loads loads) {
  constexpr int kAhead = G::kTerms == 1 ? 3 : 2;
  QFrag<G> q[kAhead];
  if (MORE)
#pragma unroll
    for (int i = 0; i < kAhead; ++i) q[i] = q_frag<G>(qnext, plane, i);
#pragma unroll
  for (int j = 0; j < G::kSteps; ++j) {
    __builtin_amdgcn_sched_barrier(0);
    if (MORE) {
      multiply_step<G, KEYS_AS_M>(j, q[j % kAhead], k, y);
      if (j + kAhead < G::kSteps) q[j % kAhead] = q_frag<G>(qnext, plane, j + kAhead);
    } else {
      loads(j);
    }
    work(j);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// All row tiles of one stage: products of the first one, then body(more, x, y, t) for every tile, the two accumulator
// sets in turn. The loads into `other` go out with the first products (here) and with the last tile (load_rest).
template <typename G, bool KEYS_AS_M, typename Body>
__device__ inline void all_row_tiles(const char* __restrict__ qrow, int plane, const Keys<G>& k, Slot<G>& other,
                                     const Pending<G>& pend, int row_tiles, Body body) {
  floatx16 xa[G::kTiles], xb[G::kTiles];
  multiply<G, KEYS_AS_M>(qrow, plane, k, xa, [&](int j) {
    __builtin_amdgcn_sched_barrier(0);
    load_some<G>(other, pend, G::kEnd + j * G::kFirst / G::kSteps, G::kEnd + (j + 1) * G::kFirst / G::kSteps);
    __builtin_amdgcn_sched_barrier(0);
  });
  int t = 0;
  for (; t + 2 < row_tiles; t += 2) {
    body(std::true_type{}, xa, xb, t);
    body(std::true_type{}, xb, xa, t + 1);
  }
  if (t + 1 < row_tiles) {
    body(std::true_type{}, xa, xb, t);
#pragma unroll
    for (int c = 0; c < G::kTiles; ++c) xa[c] = xb[c];
    ++t;
  }
  body(std::false_type{}, xa, xb, t);
}

template <typename G>
__device__ inline void load_rest(Slot<G>& other, const Pending<G>& pend, int j) {
  constexpr int from = G::kEnd + G::kFirst, n = G::kLoads - from;
  load_some<G>(other, pend, from + j * n / G::kSteps, from + (j + 1) * n / G::kSteps);
}

// Logits past the range of the products above. A split leaves NaN where an element is infinite or rounds to it, products
// of opposite sign can meet as inf - inf where multiply-adds one after the other stay on the side that overflowed first,
// and exp2(c * x - y), with c * x unrounded and y the rounded maximum or normaliser, is off by |y| 2^-25 octaves. None of
// that shows for logits of ordinary size; all of it ends as a sum of exponentials that is no number or as a |y| past
// kMaxExponent. Such sums are taken again from the elements: a row's statistics of a chunk, a key's column sum. Keys
// filled with the type's lowest value or with -inf then have no weight, as in the definition, one of several logits of
// 10^7 takes all of it, and logits of +inf or NaN leave no number in their (sequence, KV head).
// What that costs, us for 2 layers of 8192 fp32 keys of 128, 8 heads, 128 rows: 74 without, 1060 with one key in 100 of -inf
// (all rows of its chunk), 1390 with NaN in every row; the vector ALU took 570 for any.
constexpr float kMaxExponent = 8192.0f;     // logits of 5700

// Infinite or NaN (by its bits: the compiler may assume that there are no NaNs).
__device__ inline bool no_number(float v) {
  uint32_t u = __float_as_uint(v);
  asm volatile("" : "+v"(u));
  return (u & 0x7f800000u) == 0x7f800000u;
}

// y[i] = c * (logit of row i and this lane's key), as fp32 multiply-adds in the order of the elements; rounded before anything
// is subtracted from it. q: the first of eight rows, of which `rows` are there (the last one repeated for the others).
constexpr int kFmaRows = 8;
template <typename E, int D>
__device__ __forceinline__ void logits_fma(const char* __restrict__ q, int rows, const char* __restrict__ k, float c, float (&y)[kFmaRows]) {
#pragma unroll
  for (int i = 0; i < kFmaRows; ++i) y[i] = 0.0f;
#pragma unroll 4
  for (int j = 0; j < D * E::kBytes; j += 16) {
    const uint4 b = *reinterpret_cast<const uint4*>(k + j);
    const uint32_t v[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < kFmaRows; ++i) {
      const uint4 a = *reinterpret_cast<const uint4*>(q + (i < rows ? i : rows - 1) * (D * E::kBytes) + j);
      const uint32_t u[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (E::kBytes == 4) {
          y[i] = fmaf(__uint_as_float(u[e]), __uint_as_float(v[e]), y[i]);
        } else {
          y[i] = fmaf(__uint_as_float(u[e] << 16), __uint_as_float(v[e] << 16), y[i]);
          y[i] = fmaf(__uint_as_float(u[e] & 0xffff0000u), __uint_as_float(v[e] & 0xffff0000u), y[i]);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < kFmaRows; ++i) {
    y[i] *= c;
    asm volatile("" : "+v"(y[i]));
  }
}

// Column sum of a key from the elements: rows of q against the key at k, normalisers lse (log2 domain).
template <typename E, int D>
__device__ __forceinline__ float column_fma(const char* __restrict__ q, int rows, const char* __restrict__ k, float c,
                                            const float* __restrict__ lse) {
  float sum = 0.0f, y[kFmaRows];
#pragma unroll 1
  for (int r0 = 0; r0 < rows; r0 += kFmaRows) {
    logits_fma<E, D>(q + (int64_t)r0 * D * E::kBytes, rows - r0, k, c, y);
#pragma unroll
    for (int i = 0; i < kFmaRows; ++i)
      if (r0 + i < rows) sum += fast_exp2(y[i] - lse[r0 + i]);
  }
  return sum;
}

// The lower and the upper half-wavefront's value of every lane pair (l, l + 32), in both lanes.
__device__ inline void both_halves(float v, float& lower, float& upper) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  lower = __uint_as_float(h[0]);
  upper = __uint_as_float(h[1]);
}

__device__ inline const char* key_base(const TileLayers& src, const Task& t, int64_t stride_token_b, int64_t stride_head_b) {
  return src.k[t.layer] + ((int64_t)t.begin + t.c0) * stride_token_b + (int64_t)t.head * stride_head_b;
}
template <typename E>
__device__ inline const char* q_base(const TileLayers& src, const Task& t, const Params& p) {
  return src.q[t.layer] + ((int64_t)t.seq * p.Hq + (int64_t)t.head * p.G) * p.w * p.d * E::kBytes;
}

// The walk of a workgroup over its tasks and of its wavefronts over their stages, the same in both kernels: which task
// is being worked on, which comes next (its Q), whose keys are loaded when a slot is free (two stages on for bf16, the
// next task's for fp32).
template <typename E, int D, int NT>
struct Walk {
  using G = Geo<E, D, NT>;
  const TileLayers& src;
  const int32_t* __restrict__ cu;
  int64_t stride_token_b, stride_head_b;
  ChunkMap map;
  int n_seqs, Hkv, n_chunks, n_tasks, task, wave;
  Task cur, nxt;
  Slot<G> slot[G::kSlots];
  Pending<G> pend;

  __device__ Walk(const Params& p, const TileLayers& src_, const int32_t* cu_, int n_layers, int64_t st, int64_t sh)
      : src(src_), cu(cu_), stride_token_b(st), stride_head_b(sh), n_seqs(p.n_seqs), Hkv(p.Hkv) {
    map = chunk_map(cu, n_seqs, 0, 0, G::kChunk);
    n_chunks = all_chunks(cu, n_seqs, G::kChunk, map);
    n_tasks = n_chunks * Hkv * n_layers;
    task = blockIdx.x;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  }
  __device__ Task find(int i) const { return find_task(cu, n_seqs, G::kChunk, map, n_chunks, Hkv, i < n_tasks ? i : n_tasks - 1); }
  __device__ bool has_next() const { return task + (int)gridDim.x < n_tasks; }
  __device__ void expect(const Task& t, int stage, bool there) {
    // without a task to come one row is read, from the caches: the loads are issued on every path, so that the compiler's
    // count of those in flight is the same everywhere (a branch makes the other slot's waits drain them all)
    set_pending<G>(pend, key_base(src, t, stride_token_b, stride_head_b), (uint32_t)stride_token_b, stage, wave, there ? t.len : 1);
  }
  // first loads of the kernel: all of the first stage and, with two slots, the first of the second
  __device__ void begin() {
    cur = find(task);
    nxt = find(task + gridDim.x);
    expect(cur, 0, true);
    load_some<G>(slot[0], pend, 0, G::kLoads);
    if constexpr (G::kSlots == 2) {
      expect(G::kPerTask == 2 ? cur : nxt, G::kPerTask - 1, G::kPerTask == 2 || has_next());
      load_some<G>(slot[1], pend, 0, G::kEnd);
    }
  }
  // one slot: its keys have been made into operands, the next task's take their place
  __device__ void one_slot_free() { expect(nxt, 0, has_next()); }
  // two slots: slot SLOT, which held stage S of the current task, has been used up
  template <int SLOT, int S>
  __device__ void slot_used() {
    if constexpr (G::kSlots == 2) {
      if constexpr (G::kPerTask == 2) expect(nxt, S, has_next());
      else expect(find(task + 2 * gridDim.x), S, task + 2 * (int)gridDim.x < n_tasks);
      load_some<G>(slot[SLOT], pend, 0, G::kEnd);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ void advance() {
    task += gridDim.x;
    cur = nxt;
    nxt = find(task + gridDim.x);
  }
};

// stage(slot, stage of the task) for all tasks of the workgroup; the last stage of a task advances the walk.
template <typename W, typename Stage>
__device__ inline void all_stages(W& walk, Stage stage) {
  using G = typename W::G;
  while (walk.task < walk.n_tasks) {
    stage(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
    if constexpr (G::kSlots == 2) {
      if (G::kPerTask == 1 && walk.task >= walk.n_tasks) break;
      stage(std::integral_constant<int, 1>{}, std::integral_constant<int, G::kPerTask - 1>{});
    }
  }
}

// ------------------------------------------------------------------------------------------------------
// Row statistics: one partial (max, sum of exp2) per layer, chunk and row, in the log2 domain:
// y = c * x with c = softmax_scale * log2(e); partial = (max y, sum exp2(y - max y)).
// ------------------------------------------------------------------------------------------------------
template <typename E, int D, int NT>
__global__ __launch_bounds__(kThreads) void score_stats_tiles(Params p, int n_layers, TileLayers src, int64_t stride_token_b,
                                                              int64_t stride_head_b, const int32_t* __restrict__ cu,
                                                              float* __restrict__ partials, int64_t partials_stride_layer) {
  using G = Geo<E, D, NT>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int row_tiles = (p.rows + 31) >> 5, plane = row_tiles * 32 * G::kQRow;
  float2* __restrict__ stat = reinterpret_cast<float2*>(smem + G::kTerms * plane);   // [kWaves][row_tiles * 32]
  const int lane = threadIdx.x & 63;
  Walk<E, D, NT> walk(p, src, cu, n_layers, stride_token_b, stride_head_b);
  if (walk.task >= walk.n_tasks) return;
  const float cexp = p.scale * kLog2e;
  const char* __restrict__ qrow = smem + (lane & 31) * G::kQRow + (lane >> 5) * 16;
  float2* __restrict__ mine = stat + walk.wave * row_tiles * 32 + (lane & 31);
  {
    QBlock<G> q;
    load_q<G>(q, q_base<E>(src, walk.find(walk.task), p), p.rows, row_tiles);
    walk.begin();
    store_q<G>(q, smem, row_tiles);
  }
  lds_barrier();
  all_stages(walk, [&](auto slot, auto stage_of_task) {
    constexpr int SLOT = decltype(slot)::value, S = decltype(stage_of_task)::value;
    const Task& cur = walk.cur;
    Slot<G>& other = walk.slot[G::kSlots - 1 - SLOT];
    Keys<G> k;
    make_keys<G>(walk.slot[SLOT], k);
    if constexpr (G::kSlots == 1) walk.one_slot_free();
    const int prefix_rel = cur.S - p.w - cur.c0;            // first window key, relative to the chunk (may be <= 0)
    const int lim_all = prefix_rel < cur.len ? prefix_rel : cur.len;
    const int key0 = tile_key(S * G::kTiles, walk.wave);
    const bool masked = tile_key(S * G::kTiles + G::kTiles - 1, walk.wave) + 31 >= lim_all;   // a key of the stage is in the window or past the chunk
    // a quarter of the slices finds the maximum of row tile t's logits `x`, the others take the exponentials
    all_row_tiles<G, true>(qrow, plane, k, other, walk.pend, row_tiles, [&](auto more, floatx16 (&x)[G::kTiles], floatx16 (&y)[G::kTiles], int t) {
      constexpr int J = G::kSteps, JM = J / 4, V = G::kTiles * 16;
      float2 old = make_float2(-INFINITY, 0.0f);
      if (S > 0) old = mine[t * 32];
      if (masked) {
        int limit = prefix_rel + (t * 32 + (lane & 31)) % p.w;         // last key visible to this lane's row
        limit = (limit < cur.len ? limit : cur.len - 1) - key0 - 4 * (lane >> 5);
#pragma unroll
        for (int v = 0; v < V; ++v)
          if ((v >> 4) * kTileRow + 8 * ((v & 15) >> 2) + (v & 3) > limit) x[v >> 4][v & 15] = -INFINITY;
      }
      float mx = -INFINITY, m = 0.0f, m_use = 0.0f, s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
      interleave<G, true, decltype(more)::value>(qrow + (t + 1) * 32 * G::kQRow, plane, k, y, [&](int j) {
        if (j < JM) {
#pragma unroll
          for (int v = j * V / JM; v < (j + 1) * V / JM; v += 2) mx = fmaxf(mx, fmaxf(x[v >> 4][v & 15], x[v >> 4][(v & 15) + 1]));
          asm volatile("" : "+v"(mx));
          if (j == JM - 1) {
            float m_lo, m_hi;
            both_halves(mx, m_lo, m_hi);
            m = fmaxf(fmaxf(m_lo, m_hi) * cexp, old.x);
            m_use = m == -INFINITY ? 0.0f : m;
          }
        } else {
#pragma unroll
          for (int v = (j - JM) * V / (J - JM); v < (j - JM + 1) * V / (J - JM); ++v) {
            const float e = fast_exp2(fmaf(x[v >> 4][v & 15], cexp, -m_use));
            if ((v & 3) == 0) s0 += e; else if ((v & 3) == 1) s1 += e; else if ((v & 3) == 2) s2 += e; else s3 += e;
          }
          // anchored here: otherwise the compiler sinks the exponentials of all slices past the matrix instructions
          asm volatile("" : "+v"(s0), "+v"(s1), "+v"(s2), "+v"(s3));
        }
      }, [&](int j) { load_rest<G>(other, walk.pend, j); });
      float l_lo, l_hi;
      both_halves((s0 + s1) + (s2 + s3), l_lo, l_hi);
      const float l = fmaf(old.y, fast_exp2(old.x - m_use), l_lo + l_hi);
      if (lane < 32) mine[t * 32] = make_float2(m, l);
    });
    // Q of the next task (loads return in order: it arrives right behind the other slot's keys, which the next stage
    // needs anyway), then the first of the keys that take this slot
    constexpr bool kLast = S == G::kPerTask - 1;
    const bool has_next = walk.has_next();
    QBlock<G> qnext;
    if (kLast && has_next) load_q<G>(qnext, q_base<E>(src, walk.nxt, p), p.rows, row_tiles);
    walk.template slot_used<SLOT, S>();
    if (!kLast) return;
    lds_barrier();
    const int r = threadIdx.x;
    float M = -INFINITY, L = 0.0f;
    float2* __restrict__ part = reinterpret_cast<float2*>(partials + cur.layer * partials_stride_layer) +
                                ((int64_t)cur.chunk_id * p.Hkv + cur.head) * p.rows_pad;
    if (r < p.rows) {                              // the wavefronts' statistics in a fixed order
#pragma unroll
      for (int q = 0; q < kWaves; ++q) M = fmaxf(M, stat[q * row_tiles * 32 + r].x);
      const float Mu = M == -INFINITY ? 0.0f : M;
#pragma unroll
      for (int q = 0; q < kWaves; ++q) {
        const float2 v = stat[q * row_tiles * 32 + r];
        L = fmaf(v.y, fast_exp2(v.x - Mu), L);
      }
      part[r] = make_float2(M, L);
    }
    if (has_next) {
      store_q<G>(qnext, smem, row_tiles);
      lds_barrier();
    }
    // behind the barrier, where no other wavefront waits for it: rows of the chunk again, from the elements
    const bool again = no_number(L) || (M != -INFINITY && fabsf(M) > kMaxExponent);
    if (__builtin_expect(__any(again), 0)) {
      const Task t = walk.find(walk.task);         // (the current one: found again, its fields need no registers until here)
      const char* __restrict__ k0 = key_base(src, t, stride_token_b, stride_head_b);
      part = reinterpret_cast<float2*>(partials + t.layer * partials_stride_layer) + ((int64_t)t.chunk_id * p.Hkv + t.head) * p.rows_pad;
      const unsigned long long which = __ballot(again);
#pragma unroll 1
      for (int g = 0; g < 64; g += kFmaRows) {     // eight of this wavefront's rows at a time, a key to a lane
        if (!(which >> g & ((1u << kFmaRows) - 1u))) continue;
        const int r0 = walk.wave * 64 + g;
        float m[kFmaRows], l[kFmaRows], y[kFmaRows];
#pragma unroll
        for (int i = 0; i < kFmaRows; ++i) { m[i] = -INFINITY; l[i] = 0.0f; }
#pragma unroll 1
        for (int key0 = 0; key0 < t.len; key0 += 64) {
          const int key = key0 + lane;
          logits_fma<E, D>(q_base<E>(src, t, p) + (int64_t)r0 * D * E::kBytes, p.rows - r0,
                           k0 + (int64_t)(key < t.len ? key : t.len - 1) * stride_token_b, cexp, y);
#pragma unroll
          for (int i = 0; i < kFmaRows; ++i)
            if (key < t.len && key <= t.S - p.w - t.c0 + (r0 + i) % p.w) merge_pair(m[i], l[i], make_float2(y[i], 1.0f));
        }
#pragma unroll
        for (int i = 0; i < kFmaRows; ++i) {
#pragma unroll
          for (int o = 32; o > 0; o >>= 1) {
            const float2 other = make_float2(__shfl_xor(m[i], o), __shfl_xor(l[i], o));
            merge_pair(m[i], l[i], other);
          }
          if (lane == 0 && (which >> (g + i) & 1u)) part[r0 + i] = make_float2(m[i], l[i]);
        }
      }
    }
    walk.advance();
  });
}

// ---- Row normalisers lse2[row] = log2 sum_keys exp2(c * x[row, key]) from the chunk partials of the statistics
// kernel, by the kThreads threads of a workgroup: thread (row, group) of rows_pad x kThreads / rows_pad merges the
// chunks group, group + groups, ... online in chunk order into `mstage`; after a barrier thread `row` combines the
// groups. Written once and used inside the emit kernel (single-layer launches) and by the merge and export kernels
// below, so that all give the same bits.
// psrc: partials of the first chunk of this (layer, sequence, head), float2 [chunk][Hkv][rows_pad]
__device__ inline void merge_chunks(const float2* __restrict__ psrc, int n_chunks, int rows_pad, uint32_t chunk_step,
                                    float2* __restrict__ mstage) {
  const int groups = kThreads / rows_pad, row = threadIdx.x % rows_pad, group = threadIdx.x / rows_pad;
  const uint32_t t0 = (uint32_t)row + (uint32_t)group * chunk_step;   // 32-bit element offsets from a shared base
  float M = -INFINITY, Lsum = 0.0f;
#pragma unroll 8
  for (int cc = group; cc < n_chunks; cc += groups, psrc += groups * chunk_step) merge_pair(M, Lsum, psrc[t0]);
  mstage[threadIdx.x] = make_float2(M, Lsum);
}

// lse2 of row `row` (< rows_pad) from the staged merges; padding rows get +inf: exp2(x - inf) = 0
__device__ inline float combine_groups(const float2* __restrict__ mstage, int rows_pad, int row, int rows) {
  const int groups = kThreads / rows_pad;
  float M = -INFINITY;
  for (int g = 0; g < groups; ++g) M = fmaxf(M, mstage[g * rows_pad + row].x);
  const float Mu = M == -INFINITY ? 0.0f : M;
  float L = 0.0f;
  for (int g = 0; g < groups; ++g) {
    const float2 v = mstage[g * rows_pad + row];
    L = fmaf(v.y, fast_exp2(v.x - Mu), L);
  }
  return row < rows ? M + __log2f(L) : INFINITY;
}

// Merge kernel of multi-layer launches: lse_rows[layer][seq][head][rows_pad] (log2 domain), between the two
// sweeps. grid = (n_seqs, Hkv, n_layers). Inside the emit kernel this merge would sit on the critical path of every
// task (a chain of dependent loads per thread).
__global__ __launch_bounds__(kThreads) void score_merge_tiles(Params p, int chunk, const int32_t* __restrict__ cu,
                                                              const float* __restrict__ partials,
                                                              int64_t partials_stride_layer, float* __restrict__ lse_rows) {
  __shared__ float2 mstage[kThreads];
  const int seq = blockIdx.x, head = blockIdx.y, layer = blockIdx.z;
  int first = 0;
  for (int q = 0; q < seq; ++q) first += chunks_of(cu[q + 1] - cu[q], 0, chunk);
  const float2* __restrict__ psrc = reinterpret_cast<const float2*>(partials + layer * partials_stride_layer) +
                                    ((int64_t)first * p.Hkv + head) * p.rows_pad;
  merge_chunks(psrc, chunks_of(cu[seq + 1] - cu[seq], 0, chunk), p.rows_pad, (uint32_t)(p.Hkv * p.rows_pad), mstage);
  __syncthreads();
  if ((int)threadIdx.x < p.rows_pad)
    lse_rows[(((int64_t)layer * p.n_seqs + seq) * p.Hkv + head) * p.rows_pad + threadIdx.x] =
        combine_groups(mstage, p.rows_pad, threadIdx.x, p.rows);
}

// Natural-log row normalisers from the chunk partials of the statistics kernel (log2 domain):
// lse_out[(seq * Hq + head * G) * w + r]. grid = (n_seqs, Hkv).
__global__ __launch_bounds__(kThreads) void score_lse_tiles(Params p, int chunk, const int32_t* __restrict__ cu,
                                                            const float* __restrict__ partials, float* __restrict__ lse_out) {
  __shared__ float2 mstage[kThreads];
  const int seq = blockIdx.x, head = blockIdx.y;
  int first = 0;
  for (int q = 0; q < seq; ++q) first += chunks_of(cu[q + 1] - cu[q], 0, chunk);
  merge_chunks(reinterpret_cast<const float2*>(partials) + ((int64_t)first * p.Hkv + head) * p.rows_pad,
               chunks_of(cu[seq + 1] - cu[seq], 0, chunk), p.rows_pad, (uint32_t)(p.Hkv * p.rows_pad), mstage);
  __syncthreads();
  if ((int)threadIdx.x < p.rows)
    lse_out[((int64_t)seq * p.Hq + (int64_t)head * p.G) * p.w + threadIdx.x] =
        combine_groups(mstage, p.rows_pad, threadIdx.x, p.rows) * (1.0f / kLog2e);
}

// ------------------------------------------------------------------------------------------------------
// Scores: a[s] = row_scale * sum_rows exp2(c * x[row, s] - lse2[row]) over the chunk's prefix keys, max-pooled over the
// prefix. HALO (single-layer calls): the (P - 1) / 2 keys on each side of the chunk are computed as well, row tile by
// row tile spread over the wavefronts. Without (multi-layer calls): the column sums of the first and last keys of the
// chunk go to `edges`, and score_fix_borders_tiles completes the outputs next to the chunk borders.
// ------------------------------------------------------------------------------------------------------
template <typename E, int D, int NT, bool HALO>
__global__ __launch_bounds__(kThreads) void score_emit_tiles(Params p, int n_layers, TileLayers src, int64_t stride_token_b,
                                                             int64_t stride_head_b, const int32_t* __restrict__ cu,
                                                             const float* __restrict__ partials,
                                                             const float* __restrict__ lse_rows,
                                                             int64_t lse_rows_stride_layer, const float* __restrict__ lse_in,
                                                             float* __restrict__ scores, int64_t scores_stride_head,
                                                             int64_t scores_stride_layer, float* __restrict__ edges,
                                                             int64_t edges_stride_layer) {
  using G = Geo<E, D, NT>;
  using H = Geo<E, D, 1>;                                      // the halo keys: one tile
  constexpr int kChunk = G::kChunk;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int row_tiles = (p.rows + 31) >> 5, plane = row_tiles * 32 * G::kQRow;
  float* __restrict__ lse_s = reinterpret_cast<float*>(smem + G::kTerms * plane);     // [256]
  float* __restrict__ part = lse_s + 256;                                             // [kChunk + kMaxHalo], key c0 - half first
  float* __restrict__ halo_s = part + kChunk + kMaxHalo;                              // [2][8 row tiles][64] (HALO)
  float2* __restrict__ mstage = reinterpret_cast<float2*>(halo_s);                    // [kThreads] (single-layer merge)
  float* __restrict__ lse_all = halo_s + 2 * 8 * 64;                                  // [256] the normalisers as they are
  const int tid = threadIdx.x, lane = tid & 63;
  Walk<E, D, NT> walk(p, src, cu, n_layers, stride_token_b, stride_head_b);
  if (walk.task >= walk.n_tasks) return;
  const float cexp = p.scale * kLog2e;
  const int half = p.half, wave = walk.wave;
  const char* __restrict__ qrow = smem + (lane & 31) * G::kQRow + (lane >> 5) * 16;
  const float* __restrict__ lse_lane = lse_s + 4 * (lane >> 5);

  // the normaliser of row tid of a task: from lse_rows (multi-layer launches, written by the merge kernel) or lse_in
  // (supplied by the caller, natural log, single-layer launches); otherwise merged from the chunk partials
  const bool from_rows = !HALO || lse_rows != nullptr;
  auto load_normaliser = [&](const Task& t) {
    const float* __restrict__ src_row = from_rows
        ? lse_rows + (t.layer * lse_rows_stride_layer + ((int64_t)t.seq * p.Hkv + t.head) * p.rows_pad)
        : lse_in + ((int64_t)t.seq * p.Hq + (int64_t)t.head * p.G) * p.w;
    return src_row[tid < p.rows ? tid : p.rows - 1];
  };
  // lse_s: -inf in the place of normalisers past kMaxExponent, which makes every sum over their rows infinite
  auto put_normaliser = [&](float v) {                           // v: log2 domain
    if (tid < 256) {
      lse_s[tid] = tid < p.rows ? (fabsf(v) > kMaxExponent ? -INFINITY : v) : INFINITY;
      lse_all[tid] = v;
    }
  };
  auto store_normaliser = [&](float v) { put_normaliser(from_rows ? v : v * kLog2e); };
  const bool merge_here = HALO && lse_rows == nullptr && lse_in == nullptr;
  auto merge_normalisers = [&](const Task& t) {
    const int first = t.chunk_id - t.c0 / kChunk, n = (t.S + kChunk - 1) / kChunk;
    merge_chunks(reinterpret_cast<const float2*>(partials) + ((int64_t)first * p.Hkv + t.head) * p.rows_pad, n, p.rows_pad,
                 (uint32_t)(p.Hkv * p.rows_pad), mstage);
    lds_barrier();
    put_normaliser(tid < p.rows ? combine_groups(mstage, p.rows_pad, tid, p.rows) : INFINITY);
    lds_barrier();                                             // mstage and halo_s share their place
  };
  // Halo units: one row tile of one tile of halo keys (the `half` before the chunk, then the `half` behind it); the halves
  // of the rows are kept apart, for the order of summation of the other keys.
  const int halo_units = HALO ? (2 * half > 32 ? 2 : (half > 0 ? 1 : 0)) * row_tiles : 0;
  auto load_halo = [&](const Task& t, int unit, Slot<H>& kh) {
    const int e = unit / row_tiles * 32 + (lane & 31);
    int key = e < half ? e - half : kChunk + e - half;         // relative to the chunk, cut to the sequence
    key = key < t.S - t.c0 ? key : t.S - t.c0 - 1;
    key = key < -t.c0 ? -t.c0 : key;
    Pending<H> pend;
    pend.base = key_base(src, t, stride_token_b, stride_head_b) + (int64_t)key * stride_token_b + (lane >> 5) * (H::kStepBytes / 2);
    pend.off[0] = 0u;
    load_some<H>(kh, pend, 0, H::kLoads);
  };
  auto halo_unit = [&](int unit, const Slot<H>& kh) {
    const int kt = unit / row_tiles, t = unit - kt * row_tiles;
    Keys<H> k;
    make_keys<H>(kh, k);
    floatx16 acc[1];
    multiply<H, false>(qrow + t * 32 * G::kQRow, plane, k, acc, [](int) {});
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;          // in the order of the stages below
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 lz = *reinterpret_cast<const float4*>(lse_lane + t * 32 + 8 * i);
      s0 += fast_exp2(fmaf(acc[0][4 * i], cexp, -lz.x));
      s1 += fast_exp2(fmaf(acc[0][4 * i + 1], cexp, -lz.y));
      s2 += fast_exp2(fmaf(acc[0][4 * i + 2], cexp, -lz.z));
      s3 += fast_exp2(fmaf(acc[0][4 * i + 3], cexp, -lz.w));
    }
    halo_s[(kt * 8 + t) * 64 + lane] = (s0 + s1) + (s2 + s3);
  };
  auto take_again = [&](const Task& t, int key) __attribute__((always_inline)) {   // a key's sum
    return column_fma<E, D>(q_base<E>(src, t, p), p.rows, key_base(src, t, stride_token_b, stride_head_b) + (int64_t)key * stride_token_b,
                            cexp, lse_all);
  };
  {
    QBlock<G> q;
    const Task first = walk.find(walk.task);
    load_q<G>(q, q_base<E>(src, first, p), p.rows, row_tiles);
    Slot<H> kh;
    if (HALO && wave < halo_units) load_halo(first, wave, kh);
    float lse0 = 0.0f;
    if (!merge_here) lse0 = load_normaliser(first);
    walk.begin();
    store_q<G>(q, smem, row_tiles);
    if (merge_here) {
      merge_normalisers(first);
    } else {
      store_normaliser(lse0);
      lds_barrier();
    }
    if (HALO && wave < halo_units) halo_unit(wave, kh);
  }
  all_stages(walk, [&](auto slot, auto stage_of_task) {
    constexpr int SLOT = decltype(slot)::value, S = decltype(stage_of_task)::value;
    constexpr bool kLast = S == G::kPerTask - 1;
    const Task& cur = walk.cur;
    Slot<G>& other = walk.slot[G::kSlots - 1 - SLOT];
    Keys<G> k;
    make_keys<G>(walk.slot[SLOT], k);
    if constexpr (G::kSlots == 1) walk.one_slot_free();
    const int prefix = cur.S - p.w;
    int len = prefix - cur.c0;                               // prefix keys of the chunk (none: only the guard is written)
    len = len < cur.len ? len : cur.len;
    // column sums of all keys of the stage; those past the prefix are not used
    float col[G::kTiles];
#pragma unroll
    for (int c = 0; c < G::kTiles; ++c) col[c] = 0.0f;
    all_row_tiles<G, false>(qrow, plane, k, other, walk.pend, row_tiles, [&](auto more, floatx16 (&x)[G::kTiles], floatx16 (&y)[G::kTiles], int t) {
      constexpr int J = G::kSteps, T = G::kTiles, V = T * 16;
      const float* __restrict__ lse = lse_lane + t * 32;
      // value v: rows 4 (v / (4 T)) .. + 3 of the accumulators, key tile (v / 4) % T
      float4 lz = *reinterpret_cast<const float4*>(lse), lz_next = lz;
      float sum[T][4];
#pragma unroll
      for (int c = 0; c < T; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[c][e] = 0.0f;
      interleave<G, false, decltype(more)::value>(qrow + (t + 1) * 32 * G::kQRow, plane, k, y, [&](int j) {
#pragma unroll
        for (int v = j * V / J; v < (j + 1) * V / J; ++v) {
          const int g = v / (4 * T), c = (v >> 2) % T, e = v & 3;
          if (v % (4 * T) == 0) {
            lz = lz_next;
            if (g < 3) lz_next = *reinterpret_cast<const float4*>(lse + 8 * (g + 1));
          }
          const float z = e == 0 ? lz.x : (e == 1 ? lz.y : (e == 2 ? lz.z : lz.w));
          sum[c][e] += fast_exp2(fmaf(x[c][4 * g + e], cexp, -z));
        }
#pragma unroll
        for (int c = 0; c < T; ++c) asm volatile("" : "+v"(sum[c][0]), "+v"(sum[c][1]), "+v"(sum[c][2]), "+v"(sum[c][3]));   // anchored here (see the statistics)
      }, [&](int j) { load_rest<G>(other, walk.pend, j); });
#pragma unroll
      for (int c = 0; c < T; ++c) col[c] += (sum[c][0] + sum[c][1]) + (sum[c][2] + sum[c][3]);
    });
    float sums[G::kTiles];
    bool none = false;
#pragma unroll
    for (int c = 0; c < G::kTiles; ++c) {
      float lo, hi;
      both_halves(col[c], lo, hi);
      sums[c] = lo + hi;
      none |= no_number(sums[c]);
    }
    if (__builtin_expect(__any(none), 0)) {
#pragma unroll 1
      for (int c = 0; c < G::kTiles; ++c) {
        const int key = tile_key(S * G::kTiles + c, wave) + (lane & 31);
        const float had = c == 0 ? sums[0] : sums[G::kTiles - 1];
        if (key < len && no_number(had)) (c == 0 ? sums[0] : sums[G::kTiles - 1]) = take_again(cur, key);
      }
    }
#pragma unroll
    for (int c = 0; c < G::kTiles; ++c)
      if (lane < 32) part[half + tile_key(S * G::kTiles + c, wave) + lane] = sums[c] * p.row_scale;
    if (HALO && kLast)
      for (int u = wave + kWaves; u < halo_units; u += kWaves) {
        Slot<H> kh;
        load_halo(cur, u, kh);
        halo_unit(u, kh);
      }
    // as in the statistics kernel: Q and the normalisers of the next task, then the first of the keys that take this slot
    const bool has_next = walk.has_next();
    QBlock<G> qnext;
    float lse_next = 0.0f;
    if (kLast && has_next) {
      load_q<G>(qnext, q_base<E>(src, walk.nxt, p), p.rows, row_tiles);
      if (!merge_here) lse_next = load_normaliser(walk.nxt);
    }
    walk.template slot_used<SLOT, S>();
    if (!kLast) return;
    lds_barrier();
    if (HALO && half > 0) {
      if (tid < 2 * half && len > 0) {
        const int kt = tid >> 5, l = tid & 31;
        float lo = 0.0f, hi = 0.0f;
        for (int t = 0; t < row_tiles; ++t) {
          lo += halo_s[(kt * 8 + t) * 64 + l];
          hi += halo_s[(kt * 8 + t) * 64 + 32 + l];
        }
        const int key = tid < half ? tid - half : kChunk + tid - half;
        const bool in = tid < half ? cur.c0 > 0 : cur.c0 + key < prefix;   // c0 is 0 or at least a chunk, longer than half
        float sum = lo + hi;
        if (__builtin_expect(in && no_number(sum), 0)) sum = take_again(cur, key);
        part[half + key] = in ? sum * p.row_scale : -INFINITY;
      }
      lds_barrier();
    }
    // max-pool, window [i - half, i + half] cut to the keys that are there: an index clamped to the range stays inside
    // the window, and taking an element twice does not change a maximum
    float* __restrict__ out = scores + cur.layer * scores_stride_layer + (int64_t)cur.head * scores_stride_head + cur.begin + cur.c0;
    const int first = HALO && cur.c0 > 0 ? -half : 0;
    int last = HALO && len == kChunk ? kChunk + half - 1 : len - 1;
    last = last < prefix - cur.c0 - 1 ? last : prefix - cur.c0 - 1;
    if (!HALO && tid < 2 * half && len > 0) {                // [0, half): the first column sums, [half, 2 half): the last
      const int i = tid < half ? tid : len - 2 * half + tid;
      edges[cur.layer * edges_stride_layer + ((int64_t)cur.chunk_id * p.Hkv + cur.head) * kMaxHalo + tid] =
          i >= 0 && i < len ? part[half + i] : -INFINITY;
    }
#pragma unroll
    for (int u = 0; u < (kChunk + kThreads - 1) / kThreads; ++u) {
      const int i = tid + u * kThreads;
      if (i < cur.len && prefix > 0) {
        float m = -INFINITY;                                 // the guard over the window slots
        if (i < len) {
          m = part[half + i];
          for (int o = 1; o <= half; ++o) {
            const float lo = part[half + (i - o > first ? i - o : first)], hi = part[half + (i + o < last ? i + o : last)];
            m = fmaxf(m, fmaxf(lo, hi));
          }
        }
        out[i] = m;
      }
    }
    if (has_next) {
      store_q<G>(qnext, smem, row_tiles);
      if (merge_here) {
        merge_normalisers(walk.nxt);
      } else {
        store_normaliser(lse_next);
        lds_barrier();
      }
      if (HALO && wave < halo_units) {
        Slot<H> kh;
        load_halo(walk.nxt, wave, kh);
        halo_unit(wave, kh);
      }
    }
    walk.advance();
  });
}

// Completes the outputs next to the chunk borders of an emit launch that left the pooling halo out: output s of
// chunk c within `half` of the border to chunk c + 1 takes the maximum with the neighbour's column sums that its
// pooling window reaches (a maximum is exact, so the result is the one the halo variant computes).
// grid = (chunk upper bound, Hkv, layers), 64 threads: one workgroup per border, thread t < half the output
// half - t before it, thread half + u the output u after it.
__global__ __launch_bounds__(64) void score_fix_borders_tiles(Params p, int chunk, const int32_t* __restrict__ cu,
                                                              const float* __restrict__ edges, int64_t edges_stride_layer,
                                                              float* __restrict__ scores, int64_t scores_stride_head,
                                                              int64_t scores_stride_layer) {
  const ChunkMap map = chunk_map(cu, p.n_seqs, 0, 0, chunk);
  const int n_chunks = all_chunks(cu, p.n_seqs, chunk, map);
  if ((int)blockIdx.x >= n_chunks) return;
  const Task c = find_task(cu, p.n_seqs, chunk, map, n_chunks, 1, blockIdx.x);
  const int head = blockIdx.y, layer = blockIdx.z, half = p.half, t = threadIdx.x;
  const int prefix = c.S - p.w;
  const int o1 = c.c0 + chunk;                                 // first output of the next chunk
  if (t >= 2 * half || o1 >= prefix) return;
  const int next_len = o1 + chunk < prefix ? chunk : prefix - o1;
  const float* __restrict__ mine = edges + layer * edges_stride_layer + ((int64_t)blockIdx.x * p.Hkv + head) * kMaxHalo + half;
  const float* __restrict__ next = edges + layer * edges_stride_layer + ((int64_t)(blockIdx.x + 1) * p.Hkv + head) * kMaxHalo;
  float* __restrict__ out = scores + layer * scores_stride_layer + (int64_t)head * scores_stride_head + c.begin;
  float m = -INFINITY;
  int s;
  if (t < half) {            // output o1 - half + t: its window ends at o1 + t, the next chunk's first t + 1 keys
    s = o1 - half + t;
    for (int e = 0; e <= t; ++e) m = fmaxf(m, next[e]);        // -inf past the end of a short last chunk
  } else {                   // output o1 + u: its window starts at o1 + u - half, this chunk's last half - u keys
    const int u = t - half;
    if (u >= next_len) return;
    s = o1 + u;
    for (int e = u; e < half; ++e) m = fmaxf(m, mine[e]);
  }
  out[s] = fmaxf(out[s], m);
}

// Offsets of key rows inside a chunk (at most 1024 rows) are formed in 32 bits; Q has to fit LDS whole (see kMaxRows: fp32 at
// head size 128 up to 128 rows). What does not takes the vector-ALU kernels.
bool score_tiles_supported(const Params& p, int dtype, int64_t k_stride_token) {
  const int64_t stride_b = k_stride_token * (dtype == DKV_BF16 ? 2 : 4);
  if (stride_b * 1024 >= ((int64_t)1 << 32) || 2 * p.half > kMaxHalo || p.rows > 256) return false;
  return dtype == DKV_BF16 ? p.d == 64 : p.d == 64 || p.rows <= 128;
}

// Upper bound on the chunks of all sequences (the lengths are on the device: every sequence may have a ragged tail).
static int chunk_bound(const Params& p, int chunk) {
  return p.n_seqs == 1 ? (p.total_tokens + chunk - 1) / chunk : p.total_tokens / chunk + p.n_seqs;
}

// Tiles per wavefront for bf16 (1, 2 or 4: chunks of 256, 512 or 1024 keys): the count that lets one layer's tasks finish
// soonest, the larger one of two that are equal. It depends on the descriptor alone, so that a layer is cut alike
// (and gets the same bits) whether it is scored alone or with others.
static int pick_tiles(const Params& p, int cus) {
  const double fixed_us = 2.0, us_per_key = 0.0045;          // measured: 4.2 us per sweep and 1024 keys of 128 rows, 16K tokens
  int best = 4;
  double best_cost = 1e30;
  for (int nt = 4; nt >= 1; nt >>= 1) {
    const int chunk = nt * kTileRow;
    const long long rounds = ((long long)chunk_bound(p, chunk) * p.Hkv + cus - 1) / cus;
    const double cost = rounds * (fixed_us + chunk * us_per_key);
    if (cost < best_cost - 1e-9) { best_cost = cost; best = nt; }
  }
  return best;
}

constexpr int kMaxLds = 160 * 1024;

template <typename E, int D, int NT>
static hipError_t launch_tiles_t(const Params& p, int phases, int n_layers, const void* const* q_layers,
                                 const void* const* k_layers, int64_t k_stride_token, int64_t k_stride_head,
                                 const int32_t* cu, float* scores, int64_t scores_stride_head,
                                 int64_t scores_stride_layer, char* ws, const WorkspaceLayout& wl, const float* lse_in,
                                 const float* const* lse_layers, float* lse_out, hipStream_t st) {
  using G = Geo<E, D, NT>;
  constexpr int chunk = G::kChunk;
  const int cus = device_cus(), chunks = chunk_bound(p, chunk);
  float* partials = ws ? reinterpret_cast<float*>(ws + wl.partials) : nullptr;   // no workspace: lse supplied
  const int64_t partials_stride_layer = (int64_t)wl.partials_layer_bytes / (int64_t)sizeof(float);
  const int row_tiles = (p.rows + 31) / 32;
  const size_t q_bytes = (size_t)G::kTerms * row_tiles * 32 * G::kQRow;
  const size_t lds_stats = q_bytes + (size_t)kWaves * row_tiles * 32 * sizeof(float2);
  const size_t lds_emit = q_bytes + (256 + chunk + kMaxHalo + 2 * 8 * 64 + 256) * sizeof(float);
  static std::atomic<uint64_t> given{0};
  const hipError_t e = allow_lds(given, {{reinterpret_cast<const void*>(&score_stats_tiles<E, D, NT>), kMaxLds},
                                         {reinterpret_cast<const void*>(&score_emit_tiles<E, D, NT, false>), kMaxLds},
                                         {reinterpret_cast<const void*>(&score_emit_tiles<E, D, NT, true>), kMaxLds}});
  if (e != hipSuccess) return e;
  TileLayers src{};
  for (int i = 0; i < n_layers && (phases & (kPhaseStats | kPhaseEmit)); ++i) {
    src.q[i] = static_cast<const char*>(q_layers[i]);
    src.k[i] = static_cast<const char*>(k_layers[i]);
  }
  const int64_t stride_token_b = k_stride_token * E::kBytes, stride_head_b = k_stride_head * E::kBytes;
  const long long tasks = (long long)chunks * p.Hkv * n_layers;
  const unsigned grid = (unsigned)(tasks < cus ? tasks : cus);       // one workgroup per compute unit walks its tasks
  if (phases & kPhaseStats)
    launch(DKV_KERNEL_SCORE_STATS, (score_stats_tiles<E, D, NT>), dim3(grid), dim3(kThreads), lds_stats, st, p, n_layers, src,
           stride_token_b, stride_head_b, cu, partials, partials_stride_layer);
  if (phases & kPhaseEmit) {
    // The emit kernel takes the layers of the call from the last to the first: the statistics kernel has just
    // streamed them first to last, so the last layers are the ones the memory-side cache still holds.
    TileLayers rev{};
    for (int i = 0; i < n_layers; ++i) {
      rev.q[i] = src.q[n_layers - 1 - i];
      rev.k[i] = src.k[n_layers - 1 - i];
    }
    const int last = n_layers - 1;
    // several layers: their row normalisers are merged from the chunk partials by a small kernel of its own
    float* lse_rows = nullptr;
    const int64_t lse_rows_stride_layer = (int64_t)p.n_seqs * p.Hkv * p.rows_pad;
    if (n_layers > 1) {
      lse_rows = reinterpret_cast<float*>(ws + wl.lse_rows);
      if (lse_layers != nullptr)         // single sweep: the caller's normalisers, no statistics
        launch_import_lse(p, n_layers, lse_layers, lse_rows, st);
      else
        launch(DKV_KERNEL_SCORE_MERGE, score_merge_tiles, dim3(p.n_seqs, p.Hkv, n_layers), dim3(kThreads), 0, st, p, chunk, cu,
               static_cast<const float*>(partials), partials_stride_layer, lse_rows);
    } else if (lse_layers != nullptr) {
      lse_in = lse_layers[0];
    }
    // A call over several layers leaves the pooling halo to a small kernel behind the emit kernel (one launch for
    // all layers); a single layer computes the halo keys inside the emit kernel, which is cheaper than a launch.
    float* edges = n_layers > 1 ? reinterpret_cast<float*>(ws + wl.edges) : nullptr;
    const int64_t edges_stride_layer = (int64_t)wl.edges_layer_bytes / (int64_t)sizeof(float);
    auto emit = [&](auto kernel) {
      launch(DKV_KERNEL_SCORE_EMIT, kernel, dim3(grid), dim3(kThreads), lds_emit, st, p, n_layers, rev, stride_token_b,
             stride_head_b, cu, static_cast<const float*>(partials),
             lse_rows ? static_cast<const float*>(lse_rows) + last * lse_rows_stride_layer : nullptr, -lse_rows_stride_layer,
             lse_in, scores + last * scores_stride_layer, scores_stride_head, -scores_stride_layer, edges, edges_stride_layer);
    };
    if (n_layers > 1) emit(&score_emit_tiles<E, D, NT, false>);
    else emit(&score_emit_tiles<E, D, NT, true>);
    if (n_layers > 1 && p.half > 0)
      launch(DKV_KERNEL_SCORE_BORDERS, score_fix_borders_tiles, dim3(chunks, p.Hkv, n_layers), dim3(64), 0, st, p, chunk, cu,
             static_cast<const float*>(edges), edges_stride_layer, scores + last * scores_stride_layer, scores_stride_head,
             -scores_stride_layer);
  }
  if (phases & kPhaseLse)
    launch(DKV_KERNEL_SCORE_LSE, score_lse_tiles, dim3(p.n_seqs, p.Hkv), dim3(kThreads), 0, st, p, chunk, cu,
           static_cast<const float*>(partials), lse_out);
  return hipGetLastError();
}

hipError_t launch_score_tiles(const Params& p, int phases, int dtype, int n_layers, const void* const* q_layers,
                              const void* const* k_layers, int64_t k_stride_token, int64_t k_stride_head,
                              const int32_t* cu, float* scores, int64_t scores_stride_head, int64_t scores_stride_layer,
                              char* ws, const WorkspaceLayout& wl, const float* lse_in, const float* const* lse_layers,
                              float* lse_out, hipStream_t st) {
  auto go = [&](auto e, auto d, auto nt) {
    return launch_tiles_t<decltype(e), decltype(d)::value, decltype(nt)::value>(
        p, phases, n_layers, q_layers, k_layers, k_stride_token, k_stride_head, cu, scores, scores_stride_head,
        scores_stride_layer, ws, wl, lse_in, lse_layers, lse_out, st);
  };
  using I1 = std::integral_constant<int, 1>;
  using D64 = std::integral_constant<int, 64>;
  if (dtype == DKV_F32) return p.d == 64 ? go(ElemF32{}, D64{}, I1{}) : go(ElemF32{}, std::integral_constant<int, 128>{}, I1{});
  switch (pick_tiles(p, device_cus())) {
    case 1: return go(ElemBf16{}, D64{}, I1{});
    case 2: return go(ElemBf16{}, D64{}, std::integral_constant<int, 2>{});
    default: return go(ElemBf16{}, D64{}, std::integral_constant<int, 4>{});
  }
}

}  // namespace dkv
