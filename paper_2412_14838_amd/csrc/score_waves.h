// The second scoring sweep: bf16, head size 128, up to 256 score rows (G * ws) per KV head. Included by score_mfma.hip,
// whose helpers (chunks, merges, layers of a launch) it uses; the mathematics of the two sweeps is described there.
//
// A wavefront owns tiles of 32 keys and multiplies them with ALL score rows, whose Q block stays in its registers (128
// rows: 128 of 256; more: 32 for every 32 rows, accumulation registers, which matrix instructions read as an operand and nothing
// else needs, so that a SIMD holds one wavefront of 512). Its keys go from global memory straight into its own piece of LDS (global_load_lds, 16 bytes a lane)
// and from there into registers in MFMA operand layout; no other wavefront touches them, so the wavefronts of a workgroup
// need no barrier between the tiles, only three per layer. A ring of three (four) half tiles (32 keys x 64 of the head's
// dimensions, 4 KB) per wavefront is in flight. The eight (four) wavefronts take neighbouring tiles, 64 (32) KB of consecutive keys
// per round. A row of a half tile is 128 bytes, one cache line; its 16-byte pieces lie in LDS with bits 1 to 3 of the row
// folded into their place, which makes the reads (32 rows, the same piece) free of bank conflicts; the loads fold the
// same bits into the address they read from.
// A unit of work is 32 keys x 32 rows: its 8 MFMAs go out among the exponentials of the unit before it (two accumulators),
// across the ends of tiles and layers. Row tiles are unrolled, so that Q's registers have fixed names; in a layer's last
// tile the next layer's rows replace them one row tile at a time. Sums are taken in the order of score_emit_mfma: the
// scores are the same bits, whichever kernel writes them.
//
// What bounds it: up to 64 rows, the stream of keys (32 layers of 8 heads x 32768 keys in 370 us, 5.8 TB/s; a plain read 346). At
// 128 rows the issue of vector and matrix instructions: an exponential takes the SIMD 8 cycles, a plain instruction 4, an
// MFMA 8 to 10 of issue, and a second wavefront adds little to that: 320 cycles a unit at least, at a clock that falls to
// 1.5 GHz while memory streams as well.
// Against score_emit_mfma (key tiles shared by all wavefronts, a barrier every 128 keys), us, before / after:
//   32 layers, 8 heads, 32768 keys: 64 rows 409 / 370, 128 rows 470 / 420 (with the keys in the L2: 357 / 212, 375 / 311)
//   16 layers in one call, per layer, 8 heads: 65536 keys, 128 rows 29.5 / 24.8; five prompts of 4000 to 15000 keys, 64 rows
//   21.6 / 17.7, 128 rows 23.0 / 19.2; 8192 keys, 64 rows 3.74 / 3.20
//   one layer, 8 heads: 64 rows, 2048 keys 8.7 / 7.3, 16384 11.0 / 8.1, 65536 27.0 / 22.5; 128 rows, 32768 keys 18.6 / 15.9
// At 65 to 128 rows a wavefront's tile takes four units, and what a layer costs beside them shows when there are few tiles: where the
// chunk is shorter than kWvMinChunk keys score_emit_mfma stays (second sweep with the normalisers handed over, there / here: 8 layers of 64
// prompts of 300 keys, 8 heads of 128 rows 106 / 109, 96 rows 98 / 103; 4 layers of 90 to 3000 keys, 4 heads of 96 rows 17.7 / 18.4; 8 layers of 16
// prompts of 1000 keys 85 / 85). The rule does not ask for the number of layers: one layer of one sequence has no next one and would be the
// faster one here (both sweeps, 8 heads of 128 rows, 1000 keys 13.6 / 13.1, 8192 keys 15.3 / 14.7, 64 prompts of 300 keys 38.7 / 38.8).
// A batch's chunk may be cut to half of the host's on the device
// (fitted_chunk): this kernel is the faster one there all the same, before / after, 8 heads: 96 rows, 32 prompts of 30 K keys together,
// 640 of 1024 keys, one layer 32.6 / 31.8, four in one call 77.2 / 71.4; 128 rows, 16 prompts of 16 K, 768 of 1024, 15.6 / 14.2 and
// 39.4 / 34.5; 16 prompts of 45 K, 896 of 1024, 35.2 / 33.4 and 101 / 92. Up to 64 rows it is taken always, also at one tile to a
// wavefront (chunks of 256 keys): 64 rows, one layer of 300 keys 7.8 / 6.2, 8192 keys 8.6 / 6.8, eight layers in one call 31.2 / 27.1;
// 64 prompts of 300 keys, eight layers 88 / 72; 8 rows, 200 prompts of 400 keys, one layer 121 / 95.
// 129 to 256 rows: nobody else is on the SIMD, and whatever the wavefront waits for shows: its matrix instructions and exponentials
// alone take 366 cycles a unit (203 ns at the 1.8 GHz the chip holds under them), the kernel 630 (257 cycles of MFMAs, 277 of
// vector instructions). A branch around the LDS reads of the next tile would have the waits behind it, for reads of a unit ago, wait for
// those too (7 layers of 4 heads x 131072 keys, 224 rows 280 / 275). One row tile more costs what it is, not as 64 rows more for everybody.
// Against score_emit_mfma, us, before / after: 28 layers of 4 heads x 32768 keys, 224 rows 307 / 274; 16 of 2 heads x 20000, 160 rows 57 / 46
// (the same cut of the keys on both sides); with that sweep's cut of the keys, 32 of 8 heads x 8192, 256 rows 215 / 178; 8 of 4 heads x
// 4097, 192 rows 30 / 25; one layer of 4 heads x 32768, 224 rows, both sweeps 30.6 / 30.2. Normalisers kept in registers were tried and
// spill; a tile's loads one at a time between the units cost more instructions than they hide (320 us for 310 with four in a row).
// Its tiles go round the four wavefronts, 128 keys a round, and a layer's end shows, so that workgroups which take several layers through a
// short chunk are better off with score_emit_mfma and its steps of 64 keys: wide_by_shared_tiles, by the time of a layer in the longest
// chunk. Second sweep with the normalisers handed over, us, score_emit_mfma / this one: 256 rows, 100 prompts of 187 keys, 2 heads,
// 16 layers 102 / 124; 16 of 180, 8 heads, 16 layers 91 / 117; 32 of 500 to 1200, 2 heads, 32 layers 259 / 300; two of 5375 and 10801,
// 4 heads, 8 layers 69 / 80; 224 rows, 64 of 133, 2 heads, 16 layers 87 / 103, 100 of 500, 8 layers 131 / 144; 192 rows, 64 of 180, 16 layers
// 85 / 95. The other way: 256 rows, 100 of 130, 8 layers 52 / 49; 224 rows, 64 of 500, 16 layers 179 / 170, 64 of 1400 415 / 374; 192 rows,
// 64 of 90, 16 layers 86 / 69, 64 of 500 173 / 153; 160 rows, 24 of 130, 4 heads, 8 layers 53 / 43. Of 412 shapes of 129 to 256 rows, most of
// them batches, the rule's choice is the slower one by 0.17 % on average and 6 % at most; this kernel everywhere by 1.8 and 29, the other one
// by 7.2 and 35. A call of one layer always comes here: 64 prompts of 300 keys, 2 heads of 160 to 256 rows 11.3 to 12.8 / 8.6 to 10.7.
// The first sweep done the same way was not better at 128 rows (32 layers of 32768 keys 417 / 419, one layer of 8192 9.6 / 10.1),
// and its sums come out in another order.
#pragma once

namespace dkv {

constexpr int kWvHalfBytes = 4096;
constexpr int kWvMinChunk = 1024;
constexpr int wv_waves(int nrt) { return nrt > 4 ? 4 : 8; }
constexpr int wv_threads(int nrt) { return 64 * wv_waves(nrt); }
constexpr int wv_ring(int nrt) { return nrt > 4 ? 4 : 3; }         // half tiles in flight per wavefront
constexpr int wv_ring_bytes(int nrt) { return wv_waves(nrt) * wv_ring(nrt) * kWvHalfBytes; }
// Microseconds of a layer in a chunk: its end, and a step of score_emit_mfma (64 keys, at least three of them) or a round of this kernel (128
// keys); fitted to those shapes. kWvStartUs: what a workgroup of this kernel has ahead at the start.
constexpr double kStEndUs = 1.5, kStStepUs = 1.08, kWvStartUs = 1.0;
constexpr double kWvEndUs[4] = {2.25, 1.9, 2.1, 2.4}, kWvRoundUs[4] = {1.45, 1.75, 2.0, 2.1};     // 129 to 160 rows, to 192, 224, 256
// More than 128 rows: true where score_emit_mfma is the faster one for workgroups of layers_each layers and at most `keys` keys.
static bool wide_by_shared_tiles(int rows, int keys, int layers_each) {
  const int t = (rows - 129) / 32, steps = (keys + 63) / 64, rounds = (keys + 127) / 128;
  const double shared = kStEndUs + kStStepUs * (steps > 3 ? steps : 3), waves = kWvEndUs[t] + kWvRoundUs[t] * rounds;
  return layers_each * (waves - shared) > kWvStartUs;
}
// Shape of the merge of chunk partials: row slabs of 64, groups of chunks; keys per round of the wavefronts (the unit of chunks).
constexpr int wv_slabs(int nrt) { return nrt > 4 ? 4 : nrt / 2; }
constexpr int wv_groups(int nrt) { return nrt > 4 ? 2 : 4; }

// Row tiles of 32 for a call (2, 4 or 5 to 8).
__host__ __device__ constexpr int wv_rows(int nrt) { return nrt * 32; }
__host__ __device__ constexpr int wv_lse_rows(int nrt) { return (nrt + 1) / 2 * 64; }   // whole wavefronts load them
constexpr int kWvMergeBytes = 512 * (int)sizeof(float2);           // at most; merges of chunk partials share the place of the column sums
__host__ __device__ constexpr int wv_sums_bytes(int chunk) {          // column sums of a chunk: its outputs, the pooling halo, the last tile's rest
  const int b = (chunk + kMaxHalo + 32) * (int)sizeof(float);
  return b > kWvMergeBytes ? b : kWvMergeBytes;
}
template <int NRT> constexpr size_t wv_lds_emit(int chunk) {
  return wv_ring_bytes(NRT) + wv_rows(NRT) * 256 + 2 * wv_lse_rows(NRT) * sizeof(float) + wv_sums_bytes(chunk);
}

// f(0), f(1) .. f(N - 1) with the index as a constant.
template <typename F, int... I>
__device__ inline void unrolled(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ inline void unrolled(F&& f) { unrolled(f, std::make_integer_sequence<int, N>{}); }

__device__ inline uint32_t lds_address(const void* p) {
  return (uint32_t)(size_t)(__attribute__((address_space(3))) const char*)p;
}

// The lane, counted anew: where it is needed once per tile or layer it is not worth a register in between.
__device__ inline int lane_again() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// 16 (4) bytes per lane from base + off straight to LDS: lane l's land at lds + 16 l (4 l). Written as assembly because the
// compiler would put a wait for ALL loads in front of every LDS read that follows; there is no register result. Whoever
// reads the data waits with wait_newer() first. Other loads and stores of the wavefront only make that wait longer
// (they are counted in the same order). The base is copied inside: a vector instruction may have written it just before.
__device__ inline void load_lds16(uint32_t lds, uint32_t off, const char* base) {
  const char* b;
  asm volatile("s_mov_b64 %0, %3\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %0" : "=&s"(b) : "s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
__device__ inline void load_lds4(uint32_t lds, uint32_t off, const char* base) {
  const char* b;
  asm volatile("s_mov_b64 %0, %3\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %2, %0" : "=&s"(b) : "s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
// Four of the former, 1 KB apart in LDS.
__device__ inline void load_lds16x4(uint32_t lds, uint32_t off0, uint32_t off1, uint32_t off2, uint32_t off3, const char* base) {
  const char* b;
  asm volatile(
      "s_mov_b64 %0, %6\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %0\n\t"
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %0\n\t"
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %0\n\t"
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %5, %0"
      : "=&s"(b)
      : "s"(lds), "v"(off0), "v"(off1), "v"(off2), "v"(off3), "s"(base)
      : "memory", "scc", "m0");
}
// Waits until at most `n` half tiles (of four loads each) asked for last are still in flight. n is uniform.
__device__ inline void wait_newer(int n) {
  if (n >= 4) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
  else if (n == 3) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
  else if (n == 2) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  else if (n == 1) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The keys of one wavefront as a stream of half tiles: of the tiles wave, wave + WAVES, ... of the chunk, last to first, layer after
// layer. issue() asks for the next half, take() brings the oldest one into the operand registers.
template <int WAVES, int RING>
struct WaveKeys {
  char* lds;                        // of the workgroup
  uint32_t ring;                    // this wavefront's part of it
  const char* const* k_layers;      // kernel argument
  int64_t k_off;
  const char* k_ptr;                // first key of the next tile to ask for
  const char* k_layer;              // first key of the chunk in that tile's layer
  uint32_t stride_b, off[4];        // of this lane's rows 8 i + lane / 8 and piece in a half tile
  int len, wave, my_tiles;
  int layer, row0, tiles_left, issue_slot, take_slot, issued, taken, total;   // row0, tiles_left: of the next tile to ask for, in its layer; slots in bytes
  int spare;                        // the place of a half 1 that was taken waits for its refill
  uint32_t read_off[4];             // LDS places of this lane's pieces (head dimensions 16 j .. + 15) within a half

  template <int LAYERS>
  __device__ void start(char* smem, const ScoreLayers<LAYERS>& src, int64_t chunk_off, uint32_t stride, int chunk_len, int first_layer, int n_layers) {
    const int lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds = smem;
    ring = (uint32_t)(wave * (RING * kWvHalfBytes));
    k_layers = src.k;
    k_off = chunk_off;
    stride_b = stride;
    len = chunk_len;
    const int tiles = (len + 31) >> 5;
    my_tiles = tiles > wave ? (tiles - wave + WAVES - 1) / WAVES : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) off[i] = (uint32_t)(8 * i + (lane >> 3)) * stride_b + piece_off(lane, i);
    layer = first_layer;
    issue_slot = take_slot = issued = taken = 0;
    row0 = first_key(0);
    tiles_left = my_tiles;
    spare = 0;
    total = 2 * my_tiles * (n_layers - first_layer);
    k_layer = src.k[first_layer] + k_off;
    k_ptr = k_layer + (uint64_t)((uint32_t)first_key(0) * stride_b);
    const int r = lane & 31, h = lane >> 5;
#pragma unroll
    for (int j = 0; j < 4; ++j) read_off[j] = ring + (uint32_t)(r * 128 + (((2 * j + h) ^ ((r >> 1) & 7)) << 4));
  }
  // The piece that lands in place lane % 8 of row 8 i + lane / 8.
  static __device__ uint32_t piece_off(int lane, int i) { return (uint32_t)((lane & 7) ^ ((lane >> 4) + 4 * (i & 1))) * 16u; }
  __device__ int first_key(int t) const {            // of the wavefront's t-th tile, relative to the chunk
    return ((my_tiles - 1 - t) * WAVES + wave) * 32;
  }
  // The first halves: as many as the ring holds.
  __device__ void fill() {
    issue<0>();
    issue<1>();
    issue<0>();
    if (RING == 4) issue<1>();
  }
  // The next half: halves 0 and 1 in turns.
  template <int H>
  __device__ void issue() {
    if (__builtin_expect(issued >= total, 0)) return;
    const uint32_t place = lds_address(lds) + ring + (uint32_t)issue_slot;
    if (__builtin_expect(row0 + 32 <= len, 1)) {
      load_lds16x4(place, off[0], off[1], off[2], off[3], k_ptr + H * 128);
    } else {                                         // rows past the chunk repeat its last one
      const int lane = lane_again();
      uint32_t last[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        int row = row0 + 8 * i + (lane >> 3);
        row = row < len ? row : len - 1;
        last[i] = __umul24((uint32_t)row, stride_b) + piece_off(lane, i);
      }
      load_lds16x4(place, last[0], last[1], last[2], last[3], k_layer + H * 128);
    }
    ++issued;
    issue_slot = issue_slot == (RING - 1) * kWvHalfBytes ? 0 : issue_slot + kWvHalfBytes;
    if (H == 1) {
      row0 -= 32 * WAVES;
      k_ptr -= (uint64_t)(32u * WAVES * stride_b);
      if (__builtin_expect(--tiles_left == 0, 0)) {      // the wavefront's last tile of a layer
        tiles_left = my_tiles;
        ++layer;
        row0 = first_key(0);
        if (issued < total) {
          k_layer = k_layers[layer] + k_off;
          k_ptr = k_layer + (uint64_t)((uint32_t)row0 * stride_b);
        }
      }
    }
  }
  template <int H>
  __device__ void take(bf16x8 (&kf)[8]) {
    // (A wavefront alone on its SIMD reads on past the end: a branch around these reads would have every wait behind it be for them.)
    if (RING != 4 && __builtin_expect(taken >= total, 0)) return;
    if (H == 1) spare = 1;
    const int newer = issued - taken - 1;            // in the middle of the stream: RING - 1, then RING - 2
    if (__builtin_expect(newer == RING - 1 - H, 1)) {
      if (RING - 1 - H == 3) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
      else if (RING - 1 - H == 2) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    } else {
      wait_newer(newer);
    }
    const uint32_t at = (uint32_t)take_slot;
#pragma unroll
    for (int j = 0; j < 4; ++j) kf[4 * H + j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(lds + (at + read_off[j])));
    ++taken;
    take_slot = take_slot == (RING - 1) * kWvHalfBytes ? 0 : take_slot + kWvHalfBytes;
  }
  // issue() once the reads of half H have arrived: its place is the one the next half goes to. (That of half 1 is given away
  // under the exponentials that follow, in the next tile or at the end of the layer, whichever comes first.)
  template <int H>
  __device__ void refill(const bf16x8 (&kf)[8]) {
    if (H == 1) {
      if (spare == 0) return;
      spare = 0;
    }
    asm volatile("" ::"v"(kf[4 * H]), "v"(kf[4 * H + 1]), "v"(kf[4 * H + 2]), "v"(kf[4 * H + 3]) : "memory");
    issue<(H + RING) & 1>();
  }
};

// Two wavefronts share a SIMD, and the older one wins whenever both could issue: it would run ahead and wait at the next
// barrier. They have the higher priority in turns, the younger one in the first half of every tile.
__device__ inline void take_turns(int mine) {
  if (mine != 0) __builtin_amdgcn_s_setprio(1);
  else __builtin_amdgcn_s_setprio(0);
}

// The Q block of a (sequence, head): kRows rows of 256 bytes in LDS, the wavefronts fetch equal shares of them (rows past p.rows
// repeat the last one: their normalisers are +inf).
template <int NRT>
__device__ inline void load_q_block(char* qbuf, const char* q_head, int rows, int wave) {
  constexpr int kLoads = NRT * 8 / wv_waves(NRT);
  const int lane = lane_again();
#pragma unroll
  for (int i = 0; i < kLoads; ++i) {
    const int row = wave * (kLoads * 4) + 4 * i + (lane >> 4);
    const int src_row = row < rows ? row : rows - 1;
    load_lds16(lds_address(qbuf) + (uint32_t)(wave * (kLoads * 4) + 4 * i) * 256u,
               (uint32_t)src_row * 256u + (uint32_t)((lane & 15) ^ (row & 15)) * 16u, q_head);
  }
}
// Row tile t in operand layout; `at`: the places of this lane's pieces (head dimensions 16 j .. + 15) in row tile 0.
struct QPlaces {
  uint32_t at[4];                                  // the other four: ^ 128
  __device__ QPlaces() {
    const uint32_t r = threadIdx.x & 31, h = (threadIdx.x >> 5) & 1;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) at[j] = r * 256 + (((2 * j + h) ^ (r & 15)) << 4);
  }
};
__device__ inline void read_q_tile(const char* qbuf, const QPlaces& q, int t, bf16x8 (&qf)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    uint32_t at = q.at[j & 3];
    asm volatile("" : "+v"(at));                     // made anew: kept, the other four cost registers
    qf[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(qbuf + t * 8192 + (at ^ (32u * (j & 4)))));
  }
}

// More than four row tiles: Q's registers are accumulation registers, which nothing but the matrix instructions reads. Left to
// itself the compiler shares them out between both kinds and copies.
template <int NRT>
__device__ inline void keep_q_in(bf16x8 (&qf)[8]) {
  if constexpr (NRT > 4)
#pragma unroll
    for (int j = 0; j < 8; ++j) asm volatile("" : "+a"(qf[j]));
}

// The lower half-wavefront's value ([0]) and the upper half's ([1]), in every lane.
__device__ inline float2 both_halves(float v) {
  const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return make_float2(__uint_as_float(x[0]), __uint_as_float(x[1]));
}

// Scores, see score_emit_mfma (same arguments). The column sums of a chunk lie in LDS until its layer is done.
template <int NRT, int LAYERS>
__global__ __launch_bounds__(wv_threads(NRT)) void score_emit_waves(Params p, int chunk, int n_layers, int layers_each, ScoreLayers<LAYERS> src,
                                                               int64_t stride_token_b, int64_t stride_head_b,
                                                               const int32_t* __restrict__ cu, const float* __restrict__ partials,
                                                               const float* __restrict__ lse_rows, int64_t lse_rows_stride_layer,
                                                               const float* __restrict__ lse_in, float* __restrict__ scores,
                                                               int64_t scores_stride_head, int64_t scores_stride_layer,
                                                               float* __restrict__ edges, int64_t edges_stride_layer) {
  constexpr int kRows = wv_rows(NRT), kLse = wv_lse_rows(NRT), kWvThreads = wv_threads(NRT), RS = wv_slabs(NRT), KS = wv_groups(NRT);
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* qbuf = smem + wv_ring_bytes(NRT);
  float* lse_s = reinterpret_cast<float*>(qbuf + kRows * 256);           // [2][kLse] lse2 per row, by layer parity
  float* sums = lse_s + 2 * kLse;                                      // column sums by key of the chunk

  chunk = fitted_chunk(cu, p.n_seqs, chunk, Tile<RS, KS>::kKeys, gridDim.x);       // not longer than the host's: the LDS fits
  const int half = p.half;
  int seq, c, nc, begin, S, first_full, n_full;
  if (!find_chunk2(cu, p.n_seqs, p.total_tokens, chunk, p.w, blockIdx.x, seq, c, nc, begin, S, first_full, n_full)) return;
  seq = __builtin_amdgcn_readfirstlane(seq);
  begin = __builtin_amdgcn_readfirstlane(begin);
  const int head = blockIdx.y;
  const int first_layer = take_share<LAYERS>(layers_each, n_layers, lse_rows, lse_rows_stride_layer, scores, scores_stride_layer, edges, edges_stride_layer);
  const int tid = threadIdx.x;
  const int prefix = __builtin_amdgcn_readfirstlane(S - p.w);            // > 0 here
  const int o0 = __builtin_amdgcn_readfirstlane(c * chunk);              // outputs [o0, o1)
  const int o1 = o0 + chunk < prefix ? o0 + chunk : prefix;
  // keys [kbeg, kend): the outputs plus the pooling halo, inside the prefix - or, with `edges`, the outputs alone:
  // then the pooled values next to a chunk border lack the neighbour's keys, the column sums of the first and the
  // last `half` keys go to `edges`, and score_fix_borders completes those outputs afterwards
  const int halo = edges != nullptr ? 0 : half;
  const int kbeg = o0 - halo > 0 ? o0 - halo : 0;
  const int kend = o1 + halo < prefix ? o1 + halo : prefix;
  const int len = kend - kbeg;                                           // <= chunk + 2 * half
  const float cexp = p.scale * kLog2e;
  const int64_t q_off = ((int64_t)seq * p.Hq + (int64_t)head * p.G) * p.w * 256;
  const float* __restrict__ lse_seq = lse_rows + ((int64_t)seq * p.Hkv + head) * p.rows_pad;     // (multi-layer launches)

  // Tiles from the last to the first: what the statistics kernel, first to last, left in the caches
  WaveKeys<wv_waves(NRT), wv_ring(NRT)> keys;
  keys.start(smem, src, ((int64_t)begin + kbeg) * stride_token_b + (int64_t)head * stride_head_b, (uint32_t)stride_token_b, len,
             first_layer, n_layers);
  load_q_block<NRT>(qbuf, reinterpret_cast<const char*>(src.q[first_layer]) + q_off, p.rows, keys.wave);
  int at_q = 0;
  keys.fill();
  // ---- lse2[row] of the first layer; padding rows get +inf: exp2(x - inf) = 0
  float* __restrict__ lse_first = lse_s + (first_layer & 1) * kLse;
  if (lse_rows != nullptr) {
    if (tid < kRows) lse_first[tid] = lse_seq[first_layer * lse_rows_stride_layer + tid];
  } else if (lse_in != nullptr) {
    if (tid < kRows)
      lse_first[tid] = tid < p.rows ? lse_in[((int64_t)seq * p.Hq + (int64_t)head * p.G) * p.w + tid] * kLog2e : INFINITY;
  } else {
    float2* mstage = reinterpret_cast<float2*>(sums);
    const float2* psrc = reinterpret_cast<const float2*>(partials) + ((int64_t)first_full * p.Hkv + head) * p.rows_pad;
    if constexpr (NRT <= 4) {
      if (tid < KS * RS * 64) merge_chunks<RS, KS>(psrc, n_full, (uint32_t)(p.Hkv * p.rows_pad), mstage);
    } else {
      merge_chunks_both(psrc, n_full, (uint32_t)(p.Hkv * p.rows_pad), mstage);
    }
    lds_barrier();
    if (tid < kRows) lse_first[tid] = combine_groups<RS, KS>(mstage, tid, p.rows);
  }
  // the normalisers of the next layer (the first kLse / 64 wavefronts) and its Q block
  auto load_next = [&](int layer) {
    if (keys.wave < kLse / 64)
      load_lds4(lds_address(lse_s + (layer & 1) * kLse + keys.wave * 64), (uint32_t)lane_again() * 4u,
                reinterpret_cast<const char*>(lse_seq + layer * lse_rows_stride_layer + keys.wave * 64));
    load_q_block<NRT>(qbuf, reinterpret_cast<const char*>(src.q[layer]) + q_off, p.rows, keys.wave);
    at_q = keys.issued;
  };
  wait_newer(keys.issued - at_q);
  lds_barrier();
  bf16x8 qf[NRT][8], kf[8];
  const QPlaces q_places;
#pragma unroll
  for (int t = 0; t < NRT; ++t) read_q_tile(qbuf, q_places, t, qf[t]);
#pragma unroll
  for (int j = 0; j < 8; ++j) kf[j] = qf[0][j];
  keys.template take<0>(kf);
  keys.template take<1>(kf);
  if (first_layer + 1 < n_layers) {
    lds_barrier();                                                       // every wavefront has its Q: the block's place is free
    load_next(first_layer + 1);
  }
  keys.template refill<0>(kf);

  constexpr int kAccs = NRT % 2 == 0 ? 2 : 3;                            // an odd number's last one has an accumulator of its own
  floatx16 acc[kAccs];
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[kAccs - 1][e] = 0.0f;
  float4 lz[4] = {};                                                     // normalisers of a unit's rows, read from LDS a unit ahead
  int row0 = -1;                                                         // first key of the tile whose exponentials are taken; none yet
  const float* __restrict__ lse_cur = nullptr;                           // of the layer: + 32 * (row tile) + 8 * (e / 4) + e % 4
  float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f, slab = 0.0f;         // slab: of the rows before
  auto unit = [&](auto rt_c, auto mul_c) {
    constexpr int RT = decltype(rt_c)::value, PT = (RT + NRT - 1) % NRT;
    constexpr bool MUL = decltype(mul_c)::value;
    constexpr int kCur = RT == NRT - 1 ? kAccs - 1 : RT & 1, kPrev = PT == NRT - 1 ? kAccs - 1 : PT & 1;
    floatx16& cur = acc[kCur];
    floatx16& a = acc[kPrev];
    if (MUL) keep_q_in<NRT>(qf[RT]);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      __builtin_amdgcn_sched_barrier(0);
      if (RT == 0 && j == (NRT > 4 ? 6 : 2)) keys.template refill<1>(kf);
      if (MUL) {
        if (j == 0) {
          floatx16 zero;
#pragma unroll
          for (int e = 0; e < 16; ++e) zero[e] = 0.0f;
          cur = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[RT][j], kf[j], zero, 0, 0, 0);
        } else {
          cur = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[RT][j], kf[j], cur, 0, 0, 0);
        }
      }
      if ((j & 1) == 0) {
        s0 += fast_exp2(fmaf(a[2 * j], cexp, -lz[j >> 1].x));
        s1 += fast_exp2(fmaf(a[2 * j + 1], cexp, -lz[j >> 1].y));
      } else {
        s2 += fast_exp2(fmaf(a[2 * j], cexp, -lz[j >> 1].z));
        s3 += fast_exp2(fmaf(a[2 * j + 1], cexp, -lz[j >> 1].w));
        lz[j >> 1] = *reinterpret_cast<const float4*>(lse_cur + RT * 32 + 8 * (j >> 1));     // of the next unit
      }
      if (MUL && RT == NRT - 1 && j == 4) keys.template take<0>(kf);
      asm volatile("" : "+v"(s0), "+v"(s1), "+v"(s2), "+v"(s3));       // an anchor: without it the exponentials sink below all MFMAs
    }
    __builtin_amdgcn_sched_barrier(0);
    if (MUL && RT == NRT - 1) {
      keys.template take<1>(kf);
      keys.template refill<0>(kf);
    }
    if ((PT & 1) || PT == NRT - 1) {                                   // 64 rows, summed up as score_emit_mfma does: the same bits
      const float2 x = both_halves((s0 + s1) + (s2 + s3));
      s0 = s1 = s2 = s3 = 0.0f;
      slab = PT <= 1 ? x.x + x.y : slab + (x.x + x.y);
      if (PT == NRT - 1) {                                             // the tile's last rows: its column sums are complete
        const int lane = lane_again();
        if (row0 >= 0 && lane < 32) sums[row0 + lane] = row0 + lane < len ? slab * p.row_scale : -INFINITY;
      }
    }
  };
  // A layer's end, behind the first unit of the next one (no loops around global memory instructions: keys are in flight)
  auto pool_layer = [&](int li) {
    lds_barrier();                                                       // all column sums are in LDS; every wavefront has the next layer's Q
    if (li + 2 < n_layers) load_next(li + 2);
    const int tid = keys.wave * 64 + lane_again();
    if (edges != nullptr && tid < 2 * half) {                            // [0, half): the first column sums, [half, 2 half): the last
      const int i = tid < half ? tid : len - 2 * half + tid;
      edges[li * edges_stride_layer + ((int64_t)blockIdx.x * p.Hkv + head) * kMaxHalo + tid] =
          i >= 0 && i < len ? sums[i] : -INFINITY;
    }
    // max-pool, window [i - half, i + half] cut to [0, len): an index clamped to the range stays inside the window, and
    // taking an element twice does not change a maximum
    float* __restrict__ out = scores + li * scores_stride_layer + (int64_t)head * scores_stride_head + begin;
    auto pool = [&](int s0, bool two) {                                    // outputs s0 and, with `two`, s0 + kWvThreads
      const int i0 = s0 - kbeg, i1 = i0 + (two ? kWvThreads : 0);
      float m0 = sums[i0], m1 = sums[i1];
      for (int o = 1; o <= half; ++o) {
        const float a0 = sums[i0 - o > 0 ? i0 - o : 0], b0 = sums[i0 + o < len ? i0 + o : len - 1];
        const float a1 = sums[i1 - o > 0 ? i1 - o : 0], b1 = sums[i1 + o < len ? i1 + o : len - 1];
        m0 = fmaxf(m0, fmaxf(a0, b0));
        m1 = fmaxf(m1, fmaxf(a1, b1));
      }
      out[s0] = m0;
      if (two) out[s0 + kWvThreads] = m1;
    };
#pragma unroll
    for (int u = 0; u < kMaxChunk / kWvThreads; u += 2) {
      const int s = o0 + tid + u * kWvThreads;
      if (s < o1) pool(s, s + kWvThreads < o1);
    }
    if (c == nc - 1 && tid < p.w) out[prefix + tid] = -INFINITY;         // guard over the window slots (w <= 256 <= threads)
  };
  for (int li = first_layer; li < n_layers; ++li) {
    lse_cur = lse_s + (li & 1) * kLse + 4 * (lane_again() >> 5);
    for (int k = 0; k < keys.my_tiles || k == 0; ++k) {
      if (NRT <= 4) take_turns(keys.wave >> 2);
      if (keys.my_tiles > 0) unit(std::integral_constant<int, 0>{}, std::true_type{});
      if (k == 0 && li > first_layer) {
        pool_layer(li - 1);
        lds_barrier();                                                 // the column sums are read
      }
      row0 = keys.first_key(k);
      const int turn_q = (li + 1 < n_layers) & (k + 1 >= keys.my_tiles);
      if (turn_q) {                                                    // the layer's last tile: a row tile's Q gives way to the next layer's once it is used
        wait_newer(keys.issued - at_q);
        lds_barrier();
        read_q_tile(qbuf, q_places, 0, qf[0]);
      }
      if (keys.my_tiles == 0) break;
      unrolled<NRT - 1>([&](auto i) {
        constexpr int RT = decltype(i)::value + 1;
        if (NRT <= 4 && RT == NRT / 2) take_turns((keys.wave >> 2) ^ 1);
        unit(std::integral_constant<int, RT>{}, std::true_type{});
        if (turn_q) read_q_tile(qbuf, q_places, RT, qf[RT]);
      });
    }
  }
  if (keys.my_tiles > 0) unit(std::integral_constant<int, 0>{}, std::false_type{});
  pool_layer(n_layers - 1);
}

}  // namespace dkv
