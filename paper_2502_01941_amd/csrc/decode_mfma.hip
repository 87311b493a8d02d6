// Split-KV decode attention with the logits on the matrix cores
// (Section 5.1, Eq. 7 and 9: attention of the current query over prefill rows and decode slots).
//
// A workgroup owns one token range of one (sequence, KV head).  The range is cut into blocks of 4 KB of rows, dealt to
// its four waves in turn, and every wave makes two passes over its own blocks without waiting for the others, in pieces
// of as many as the logit buffer holds (more than one piece only in the LONG form):
//   1. K pass: the logits of 4 or 8 tokens per matrix step, with the head dimension cut into pieces that
//      sit in different operand rows/columns, so that the A operands are whole K rows fetched straight
//      from global memory with coalesced 16-byte loads (RowShape), two blocks in flight or in use.  The scaled logits go
//      to the wave's part of the LDS buffer, their maximum stays in registers.
//   between: weights 2^(z - reference), the wave's own maximum rounded up, tokens along the lanes; decode-slot logits are also
//      written out for the retention score (Eq. 7).  The first V rows are already on their way: they are requested ahead
//      of the use of a wave's last K blocks.
//   2. V pass: RowShape::kLanes lanes stream one V row each (16 bytes per lane) and accumulate weight * V with
//      the weights read from LDS, the next block in flight while one is used.  No rescaling is needed within a piece
//      because the maximum is already known.
// At the end the waves' sums are scaled to their common reference and added through LDS.
// Bound by the stream of K and V rows.  32 query / 8 KV heads, head_dim 128 bf16, ~5100 rows, whole steps with waves that
// wait for each other between the passes (8 KB blocks, one in flight) and with this: 16 sequences 66.1 and 64.3 us, 24
// 101.2 and 96.7; 3 sequences of 5500 rows and 5 query heads per KV head 31.3 and 28.2; 2 of 1760 rows of head_dim 64 18.6
// and 17.0 (short ranges: 8 KB blocks leave waves idle in the V pass, 19.4); one of 3790 rows 17.2 and 17.0.  512
// sequences in one launch: see decode_whole.  A microbenchmark of the same reads reaches 7.0 TB/s, this 6.6 there.
#include "common.hpp"

#include <type_traits>

namespace shotkv {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(4))) float floatx4;

// 16 bytes of a K or V row with the non-temporal hint.  A step reads every live row once; once the caches
// of a batch outgrow L2 and the memory-side cache, rows that do not settle there stream faster (4-7 %
// at 16 and more sequences of 5K tokens, no change for one to four sequences).
template <typename V>
__device__ __forceinline__ V stream_load(const char* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
}

// Buffer loads: no stride, byte offsets checked against the size (zeros past it), 32-bit data.
constexpr int kBufferFlags = 0x00027000;
constexpr int kNonTemporal = 2;  // of a buffer load's cache policy
constexpr int kOutOfBounds = 1 << 30;  // an offset past every buffer here

// value of the lane N places away inside each row of 16 lanes (rotation, so every lane gets one)
template <int N>
__device__ __forceinline__ float row_rotate(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 | N, 0xf, 0xf, false));
}

// Sums over the lanes that differ in bit 5 and, for rows of 16 lanes or fewer, 4 and 3 of the lane number, of N values per
// lane, with half of the values left to each side of an exchange: an exchange adds two values at a time.  On return
// x[0 .. kSumParts) are the sums of values kSumParts * part .. of the lane's `part`.
template <int LANES, int N> constexpr int kSumParts = LANES == 32 ? N / 2 : N / 4;
template <int LANES>
__device__ __forceinline__ int sum_part(int lane) {
  return LANES == 32 ? lane >> 5 : 2 * (lane >> 5) + ((lane >> 4) & 1);
}
template <int LANES, int N>
__device__ __forceinline__ void sum_scatter(float (&x)[N]) {
  auto add = [](const auto& r) { return __uint_as_float(r[0]) + __uint_as_float(r[1]); };
#pragma unroll
  for (int i = 0; i < N / 2; ++i)
    x[i] = add(__builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[i + N / 2]), false, false));
  if constexpr (LANES <= 16)
#pragma unroll
    for (int i = 0; i < N / 4; ++i)
      x[i] = add(__builtin_amdgcn_permlane16_swap(__float_as_uint(x[i]), __float_as_uint(x[i + N / 4]), false, false));
  if constexpr (LANES == 8)
#pragma unroll
    for (int i = 0; i < N / 4; ++i) x[i] += row_rotate<8>(x[i]);
}

// Lanes of a wave exchange values through LDS: a wave's LDS instructions run in order, so the compiler must keep theirs.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// 2^(z - reference) of a whole reference, with a mantissa that z alone decides: z - reference is rounded at another place for
// every reference, so equal logits of waves with different maxima would get weights that differ in the last bit.
__device__ __forceinline__ float exp2_of_whole_reference(float z, float reference) {
  const float top = fmaxf(ceilf(z), -0x1p30f);  // (minus infinity: no weight)
  const float up = __builtin_amdgcn_fmed3f(top - reference, -1024.f, 1024.f);
  return __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(z - top), static_cast<int>(up));
}

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kMaxRange = kDecodeMaxRange;  // tokens whose logits the LDS buffer holds at a time
constexpr int kBlockLoads = kDecodeBlockBytes / 1024;  // load instructions per block of rows

// How a row lies across the lanes of the K pass.  A matrix step has 16 operand rows and 16 columns and four
// k-slices of 16 bytes (lane / 16).  A's row holds piece `i % kPieces` of token `i / kPieces`, B's column
// j = kCols * piece + h the same piece of query head h, so C[kPieces * tau + piece][kCols * piece + h] is that
// piece's share of the logit and the shares of one logit sit in lanes kCols apart.  Laid out like this the
// lanes that hold one token read its whole row (256 bytes of it per load) with one 16-byte load each.
template <int ROW_BYTES> struct RowShape {
  static constexpr int kPieces = ROW_BYTES == 128 ? 2 : 4;
  static constexpr int kCols = 16 / kPieces;                        // query heads per matrix step
  static constexpr int kTokens = 16 / kPieces;                      // tokens per matrix step
  static constexpr int kLoads = ROW_BYTES * kTokens / (kWave * 16); // 1 KB loads per matrix step
  static constexpr int kBlock = kDecodeBlockBytes / ROW_BYTES;      // tokens a wave takes at a time
  static constexpr int kLanes = ROW_BYTES / 16;                     // lanes per row in the V pass
};

template <typename T> struct Operand;  // 16 bytes of a row as one lane holds them
template <> struct Operand<bf16_t> { typedef bf16x8 Vec; };
template <> struct Operand<float> { typedef floatx4 Vec; };
// The shares of a step's logits from its loads.  fp32 sums the four elements of a lane's 16 bytes apart and adds the four
// sums at the end: a fourth of the roundings in a row, and four chains of matrix instructions instead of one.
template <int LOADS>
__device__ __forceinline__ floatx4 multiply_step(const bf16x8* a, const bf16x8 (&b)[LOADS]) {
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < LOADS; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j], b[j], acc, 0, 0, 0);
  return acc;
}
template <int LOADS>
__device__ __forceinline__ floatx4 multiply_step(const floatx4* a, const floatx4 (&b)[LOADS]) {
  floatx4 acc[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    acc[e] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < LOADS; ++j) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j][e], b[j][e], acc[e], 0, 0, 0);
  }
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

template <typename T> struct Widen;   // the elements of 16 bytes as floats
template <> struct Widen<bf16_t> {
  static constexpr int kElems = 8;
  __device__ static void get(const u32x4& raw, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(raw[i] << 16);
      f[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
    }
  }
};
template <> struct Widen<float> {
  static constexpr int kElems = 4;
  __device__ static void get(const u32x4& raw, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(raw[i]);
  }
};

// LONG: ranges of more than kMaxRange tokens, taken in pieces of about as many.  whole (LONG only): the range is all of a
// sequence; the workgroup writes the attention output itself and, to z_dec, one partial score per slot and KV head.
template <typename T, int D, int G, bool LONG>
__global__ __launch_bounds__(kThreads, (G == 8 ? 3 : 4) - LONG) void decode_partial_kernel(
    const char* __restrict__ k_prefill, const char* __restrict__ v_prefill,
    const int32_t* __restrict__ prefill_count, char* __restrict__ k_dec, char* __restrict__ v_dec,
    const int32_t* __restrict__ slot_pos, int cap, int n_slots, int H, int H_kv, int n_group,
    int n_splits, int split_tokens, int ahead_slots, float scale_log2e, const char* __restrict__ q_new,
    const char* __restrict__ k_new, const char* __restrict__ v_new, float2* __restrict__ part_ml,
    float* __restrict__ part_o, float* __restrict__ z_dec, int32_t* __restrict__ new_slot_out, bool whole) {
  constexpr int kRow = D * static_cast<int>(sizeof(T));  // bytes per row
  if (!LONG || G == 1 || (G == 8 && kRow > 128)) whole = false;  // (decode_whole)
  typedef RowShape<kRow> S;
  constexpr int E = Widen<T>::kElems;
  const int split = blockIdx.x, g = blockIdx.y, s = blockIdx.z;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);

  constexpr int kRowsPerLoad = kWave / S::kLanes;  // V rows of one load instruction
  static_assert(kRowsPerLoad * kBlockLoads == S::kBlock && kBlockLoads % S::kLoads == 0, "whole loads and steps");
  // A wave's logits, then its weights, then its output sums: the blocks of a piece - its live prefill rows, then its
  // slots, each padded to whole blocks - are dealt to the waves in turn.
  constexpr int kMapRows = decode_map_rows(kRow), kOwnRows = kMapRows / kWaves;
  static_assert(kWaves == 4 && kOwnRows % S::kBlock == 0, "whole blocks for four waves");
  __shared__ __attribute__((aligned(16))) float zbuf[kWaves][kOwnRows][G];
  __shared__ float s_max[kWaves][G];
  __shared__ float s_sum[kWaves][G];
  static_assert(D <= kOwnRows, "output sums fit");
  __shared__ int s_red[2][kWaves];
  __shared__ int s_sp[kMapRows + S::kBlock];  // slot map of the decode slots of the piece, and what nothing depends on

  // G is the group size rounded up to a power of two; heads past the real n_group are zero queries
  // whose results are never written
  const size_t head0 = static_cast<size_t>(s) * H + static_cast<size_t>(g) * n_group;
  const int i16 = lane & 15, ksl = lane >> 4;          // A row / B column, and k-slice of the lane
  const int tau = i16 / S::kPieces;                    // as A row: token of the step
  const int col_piece = i16 / S::kCols, col_head = i16 % S::kCols;  // as B/C column
  const int a_off = 64 * (i16 % S::kPieces) + 16 * ksl;             // byte offset inside (each 256 bytes of) a row
  constexpr int kHeadSets = (G + S::kCols - 1) / S::kCols;
  typedef typename Operand<T>::Vec Vec;
  Vec bq[kHeadSets][S::kLoads];
#pragma unroll
  for (int m = 0; m < kHeadSets; ++m)
#pragma unroll
    for (int j = 0; j < S::kLoads; ++j) {
      u32x4 raw = {0u, 0u, 0u, 0u};
      const int hq = col_head + S::kCols * m;
      if (hq < n_group)
        raw = *reinterpret_cast<const u32x4*>(q_new + (head0 + hq) * kRow + 256 * j + 64 * col_piece + 16 * ksl);
      bq[m][j] = __builtin_bit_cast(Vec, raw);
    }
  // Token axis of a sequence: t < cap is row t of the prefill cache (live while t < prefill_count), t >= cap is
  // decode slot t - cap.  A range is a part of the one followed by a part of the other; every block of rows lies
  // in one part, so its address is a wave-uniform base plus a small lane offset.
  const int32_t* sp = slot_pos + static_cast<size_t>(s) * n_slots;
  const int pc = min(prefill_count[s], cap);
  const int range_begin = split * split_tokens;
  const int range_end = min(range_begin + split_tokens, cap + n_slots);
  const size_t plane = static_cast<size_t>(s) * H_kv + g;
  const char* kp = k_prefill + plane * cap * kRow;
  const char* vp = v_prefill + plane * cap * kRow;
  char* kd = k_dec + plane * n_slots * kRow;
  char* vd = v_dec + plane * n_slots * kRow;
  const char* kn = k_new + plane * kRow;
  const char* vn = v_new + plane * kRow;

  // ---- K rows: block [row0, row0 + kBlock) of the `rows` rows that start at `base`.  For rows past the end the buffer's
  // bounds check returns zeros; their logits are not used. ------------------------------------------------------------
  constexpr int kStepsPerBlock = kBlockLoads / S::kLoads;
  Vec kraw[2][kBlockLoads];  // the wave's next two blocks
  auto load_block = [&](const char* base, int row0, int rows, Vec (&raw)[kBlockLoads]) __attribute__((always_inline)) {
    char* at = const_cast<char*>(base) + static_cast<size_t>(row0) * kRow;
    // (a block may lie behind the last row: never a negative size, which would be an unbounded one)
    const auto block = __builtin_amdgcn_make_buffer_rsrc(at, 0, min(max(rows - row0, 0), S::kBlock) * kRow, kBufferFlags);
    int off = tau * kRow + a_off;
    asm("" : "+v"(off));
#pragma unroll
    for (int i = 0; i < kBlockLoads; ++i)
      raw[i] = __builtin_bit_cast(
          Vec, __builtin_amdgcn_raw_buffer_load_b128(
                   block, off + (i / S::kLoads) * S::kTokens * kRow + (i % S::kLoads) * 256, 0, kNonTemporal));
  };
  // A wave's first blocks are requested before the count of live rows has arrived (dead rows may hold anything).
  const int early_rows = min(range_end, cap) - range_begin;
#pragma unroll
  for (int j = 0; j < 2; ++j)
    if ((wave + j * kWaves) * S::kBlock < early_rows)
      load_block(kp + static_cast<size_t>(range_begin) * kRow, (wave + j * kWaves) * S::kBlock, early_rows, kraw[j]);
  // Only a range that reaches into the decode slots needs the slot that takes the new token, the lowest free
  // one, and the slot map of its (first) piece with the last occupied slot of it (a pool that is still filling
  // up is empty behind that); all come out of one round of loads.
  // A range of nothing but slots does not wait for the map with a wave's first K blocks if they begin among the first
  // ahead_slots slots (ahead_of_map); whole blocks are requested, and a wave whose block was not requested asks for it
  // when the map is there.  A free slot may hold anything: its logits are not used, and the new token's row replaces what
  // its slot held.
  const int early_slots =
      !LONG && range_begin >= cap ? min(range_end - range_begin, ahead_slots - (range_begin - cap)) : 0;
  int new_slot = n_slots, last_used = -1;
  if (range_end > cap) {
    constexpr int kBatch = 8;  // loads in flight per thread
    const int d_lo = max(range_begin - cap, 0), d_hi = range_end - cap;
    int best = INT32_MAX;
    int pos[kBatch];
    auto load_map = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < kBatch; ++j) pos[j] = sp[min(i0 + j * kThreads, n_slots - 1)];
    };
    load_map(tid);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if ((wave + j * kWaves) * S::kBlock < early_slots)  // behind the map, as loads return in order
        load_block(kd + static_cast<size_t>(range_begin - cap) * kRow, (wave + j * kWaves) * S::kBlock,
                   range_end - range_begin, kraw[j]);
#pragma clang loop unroll(disable)
    for (int i0 = tid; i0 < n_slots && (best == INT32_MAX || i0 < d_hi); i0 += kBatch * kThreads) {
      if (i0 != tid) load_map(i0);
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const int i = min(i0 + j * kThreads, n_slots - 1);
        if (pos[j] < 0) best = min(best, i);
        if (i >= d_lo && i < d_hi) {
          if (!LONG || i - d_lo < kMapRows) s_sp[i - d_lo] = pos[j];
          if (pos[j] >= 0) last_used = max(last_used, i);
        }
      }
    }
    best = wave_min(best);
    last_used = wave_max(last_used);
    if (lane == 0) { s_red[0][wave] = best; s_red[1][wave] = last_used; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      best = min(best, s_red[0][w]);
      last_used = max(last_used, s_red[1][w]);
    }
    new_slot = __builtin_amdgcn_readfirstlane(best == INT32_MAX ? -1 : best);
    if (new_slot < d_hi) last_used = max(last_used, new_slot);
    last_used = __builtin_amdgcn_readfirstlane(last_used);
  }
  if (range_end == cap + n_slots && g == 0 && tid == 0) new_slot_out[s] = new_slot;

  float (*zown)[G] = zbuf[wave];
  // Of this wave's tokens: the largest logits, this lane's share of the sums of weights, and its part of the output sums,
  // elements kOwnSums * sum_part() .. of the [G][E] that lanes of the same columns hold together.
  constexpr int kOwnSums = kSumParts<S::kLanes, G * E>;
  float M[G], L[G], sums[kOwnSums];
#pragma unroll
  for (int h = 0; h < G; ++h) { M[h] = -INFINITY; L[h] = 0.f; }
#pragma unroll
  for (int j = 0; j < kOwnSums; ++j) sums[j] = 0.f;

  const int n_p = max(min(range_end, pc) - range_begin, 0);  // live prefill rows of the range
  const int d_lo = max(range_begin - cap, 0);                // its decode slots: [d_lo, d_lo + n_d)
  const int n_d = max(min(range_end - cap, last_used + 1) - d_lo, 0);
  const int new_row = new_slot >= d_lo && new_slot < d_lo + n_d ? new_slot - d_lo : -1;  // the new token's, if inside
  const char* kp0 = kp + static_cast<size_t>(range_begin) * kRow;
  const char* vp0 = vp + static_cast<size_t>(range_begin) * kRow;
  char* kd0 = kd + static_cast<size_t>(d_lo) * kRow;
  char* vd0 = vd + static_cast<size_t>(d_lo) * kRow;
  // The blocks of the range: prefill rows, then slots; dealt to the waves in turn.  The slots of a whole sequence start a
  // piece of their own, so that their weights are all still there when the sums are known.
  int nb_p = ceil_div(n_p, S::kBlock);
  if (whole) nb_p = ceil_div(nb_p, kWaves) * kWaves;
  const int n_blk = new_slot >= 0 ? nb_p + ceil_div(n_d, S::kBlock) : 0;
  int b0 = 0, b1 = 0, map0 = 0;  // the blocks of the piece, the first slot of the slot map
  if (n_blk > 0)
#pragma clang loop unroll(disable)
    for (;; b0 = b1) {
      const bool first = !LONG || b0 == 0;
      // In a loop the compiler keeps what it can derive from the lane number in registers through it: made anew here.
      int lane = threadIdx.x % kWave;
      if (LONG) asm volatile("" : "+v"(lane));
      const int i16 = lane & 15, ksl = lane >> 4, tau = i16 / S::kPieces;
      const int col_piece = i16 / S::kCols, col_head = i16 % S::kCols, a_off = 64 * (i16 % S::kPieces) + 16 * ksl;
      const int grp = lane / S::kLanes, v_off = 16 * (lane % S::kLanes);
      b1 = n_blk;
      if (LONG) b1 = min(b1, b0 < nb_p && whole ? min(b0 + kWaves * kOwnRows / S::kBlock, nb_p) : b0 + kWaves * kOwnRows / S::kBlock);
      if (LONG && n_d > kMapRows) {
        __syncthreads();  // the previous piece's slot map is done with
        map0 = max(b0 - nb_p, 0) * S::kBlock;
        for (int i = tid; i < kMapRows; i += kThreads)
          if (map0 + i < n_d) s_sp[i] = sp[d_lo + map0 + i];
        __syncthreads();
      }
      auto slot_used = [&](int i) __attribute__((always_inline)) {
        return (i == new_row || s_sp[i - map0] >= 0) && i < n_d;
      };

      // ---- pass 1: logits --------------------------------------------------------------------------------
      float mx[kHeadSets];  // largest logit this lane has seen, of head col_head + kCols * m
#pragma unroll
      for (int m = 0; m < kHeadSets; ++m) mx[m] = -INFINITY;
      auto append = [&](int row0, Vec (&raw)[kBlockLoads]) __attribute__((always_inline)) {
        if (new_row >= row0 && new_row < row0 + S::kBlock) {  // only this workgroup reads the slot this step
#pragma unroll
          for (int i = 0; i < kBlockLoads; ++i)
            if (row0 + (i / S::kLoads) * S::kTokens + tau == new_row) {
              raw[i] = stream_load<Vec>(kn + (i % S::kLoads) * 256 + a_off);
              *reinterpret_cast<Vec*>(kd0 + static_cast<size_t>(new_row) * kRow + (i % S::kLoads) * 256 + a_off) = raw[i];
            }
        }
      };
      auto fetch = [&](int blk, Vec (&raw)[kBlockLoads]) __attribute__((always_inline)) {
        if (blk < nb_p) {
          load_block(kp0, blk * S::kBlock, n_p, raw);
          return;
        }
        // A slot without a token is given an offset out of bounds, so it is zeros and costs no traffic, as in the V pass
        // (every other slot of 1025 free: 58.7 us a step for 16 caches of 4000 rows, 60.8 with all slots fetched).  A
        // block requested ahead of the map has its free slots fetched.
        const int row0 = (blk - nb_p) * S::kBlock;
        char* at = kd0 + static_cast<size_t>(row0) * kRow;
        const auto rows =
            __builtin_amdgcn_make_buffer_rsrc(at, 0, min(max(n_d - row0, 0), S::kBlock) * kRow, kBufferFlags);
        const int* map = s_sp + (row0 - map0) + tau;
#pragma unroll
        for (int i = 0; i < kBlockLoads; ++i) {
          const bool used = map[(i / S::kLoads) * S::kTokens] >= 0;
          int off = used ? tau * kRow + a_off : kOutOfBounds;
          asm("" : "+v"(off));  // the constant goes into the instruction, not into both sides of the choice
          raw[i] = __builtin_bit_cast(
              Vec, __builtin_amdgcn_raw_buffer_load_b128(
                       rows, off + (i / S::kLoads) * S::kTokens * kRow + (i % S::kLoads) * 256, 0, kNonTemporal));
        }
        append(row0, raw);
      };
      // Logits of a block to zown[z0..]; counts(row, z): what the row at z0 + row adds to the maximum.
      auto multiply_block = [&](int z0, const Vec (&raw)[kBlockLoads], auto counts) __attribute__((always_inline)) {
#pragma unroll
        for (int st = 0; st < kStepsPerBlock; ++st) {
#pragma unroll
          for (int m = 0; m < kHeadSets; ++m) {
            const floatx4 acc = multiply_step<S::kLoads>(&raw[st * S::kLoads], bq[m]);
            const int hq = col_head + S::kCols * m;
            // this lane's column holds piece col_piece; rows 4*ksl + v are (token, piece) pairs
            constexpr int kOwn = 4 / S::kPieces;  // tokens among a lane's four rows
#pragma unroll
            for (int i = 0; i < kOwn; ++i) {
              float z;
              if constexpr (S::kPieces == 4) {
                z = col_piece == 0 ? acc[0] : col_piece == 1 ? acc[1] : col_piece == 2 ? acc[2] : acc[3];
                z += row_rotate<4>(z);
              } else {
                z = col_piece ? acc[2 * i + 1] : acc[2 * i];
              }
              z += row_rotate<8>(z);  // now every lane of the column set that shares a head has the logit
              z *= scale_log2e;
              const int row = st * S::kTokens + kOwn * ksl + i;
              mx[m] = fmaxf(mx[m], counts(row, z));
              if (i16 < S::kCols && hq < G) zown[z0 + row][hq] = z;
            }
          }
        }
      };
      auto use_block = [&](int blk, const Vec (&raw)[kBlockLoads]) __attribute__((always_inline)) {
        const int z0 = (blk - b0) / kWaves * S::kBlock;
        if (blk < nb_p) {
          // (a first block that was requested early holds dead rows behind the live ones)
          const int live = n_p - blk * S::kBlock;
          multiply_block(z0, raw, [&](int row, float z) { return row < live ? z : -INFINITY; });
        } else {
          const int row0 = (blk - nb_p) * S::kBlock;
          multiply_block(z0, raw, [&](int row, float z) { return slot_used(row0 + row) ? z : -INFINITY; });
        }
      };
      // Two blocks are in flight or in use.  A wave's first two of the first piece are there already if they lie among the
      // live rows, or were requested ahead of the slot map.
      int blk = b0 + wave;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int b = blk + j * kWaves;
        if (b >= b1) break;
        if (first && b * S::kBlock < early_slots) append(b * S::kBlock, kraw[j]);
        else if (!(first && b * S::kBlock < n_p)) fetch(b, kraw[j]);
      }
#pragma clang loop unroll(disable)
      for (; blk + 2 * kWaves < b1; blk += 2 * kWaves) {
        use_block(blk, kraw[0]);
        fetch(blk + 2 * kWaves, kraw[0]);
        use_block(blk + kWaves, kraw[1]);
        if (blk + 3 * kWaves < b1) fetch(blk + 3 * kWaves, kraw[1]);
      }

      // V rows of block b, a live prefill row or slot each; for rows past the end the buffer's bounds
      // check returns zeros, at the price of a descriptor (a live row in their place, read
      // again, could be infinite: zero times that; 16 caches of 5121 rows 68.8 us that way, 69.4 like this, 70.8 with
      // the rows cleared after the load)
      u32x4 vraw[2][kBlockLoads];
      auto load_rows = [&](int b, u32x4 (&raw)[kBlockLoads]) __attribute__((always_inline)) {
        const bool in_p = b < nb_p;
        const int row0 = (in_p ? b : b - nb_p) * S::kBlock;
        char* at = const_cast<char*>(in_p ? vp0 : vd0) + static_cast<size_t>(row0) * kRow;
        const int left = b < b1 ? min(max((in_p ? n_p : n_d) - row0, 0), S::kBlock) : 0;
        const auto rows = __builtin_amdgcn_make_buffer_rsrc(at, 0, left * kRow, kBufferFlags);
        const int* map = s_sp + (in_p ? 0 : min(row0 - map0, kMapRows)) + grp;
#pragma unroll
        for (int u = 0; u < kBlockLoads; ++u) {
          const bool used = in_p | (map[u * kRowsPerLoad] >= 0);  // (no branch: the sums before would move behind it)
          int off = used ? grp * kRow + v_off : kOutOfBounds;
          asm("" : "+v"(off));
          raw[u] = __builtin_amdgcn_raw_buffer_load_b128(rows, off + u * kRowsPerLoad * kRow, 0, kNonTemporal);
        }
      };
      const int new_blk = nb_p + new_row / S::kBlock;
      const bool takes_new = new_row >= 0 && new_blk % kWaves == wave && (!LONG || (new_blk >= b0 && new_blk < b1));
      u32x4 v_of_new = {0u, 0u, 0u, 0u};
      if (takes_new) v_of_new = stream_load<u32x4>(vn + v_off);
      // in flight while the last logits and the weights are computed
      if (blk < b1) {
        load_rows(b0 + wave, vraw[0]);
        use_block(blk, kraw[0]);
        if (blk + kWaves < b1) use_block(blk + kWaves, kraw[1]);
      }

      // ---- between the passes: maximum, weights and their sum -----------------------------------------
      // Every wave takes the values of the tokens whose logits it took, so no wave waits for another one here: the exchange
      // through LDS is between lanes, in the order of a wave's instructions.
      wave_lds_fence();
      float ref[G], alpha[G];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        // lanes 16, 32 and 48 away hold other tokens of the same head (and so do, redundantly, the other pieces)
        const int m = h / S::kCols;
        if (h % S::kCols == 0) {
          const float w = max_across_halves(mx[m]);
          const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(w), __float_as_uint(w), false, false);
          mx[m] = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
        }
        // (rounded up to a whole number: what moves sums from one reference to another is then a power of two, and exact)
        const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mx[m]), h % S::kCols));
        const float m_new = fmaxf(M[h], ceilf(w));
        alpha[h] = 0.f;
        if (LONG && M[h] != -INFINITY) {  // what earlier pieces gave moves to the new maximum
          alpha[h] = __builtin_amdgcn_exp2f(M[h] - m_new);
          L[h] *= alpha[h];
        }
        M[h] = m_new;
        ref[h] = m_new == -INFINITY ? 0.f : m_new;
      }
      const int own_rows = b0 + wave < b1 ? ((b1 - 1 - b0 - wave) / kWaves + 1) * S::kBlock : 0;
      auto take_weights = [&](auto scores_c) __attribute__((always_inline)) {
#pragma clang loop unroll(disable)
        for (int t = lane; t < own_rows; t += kWave) {
          const int b = b0 + wave + t / S::kBlock * kWaves, row = b * S::kBlock + t % S::kBlock;
          const int slot = row - nb_p * S::kBlock;
          const bool valid = slot < 0 ? row < n_p : slot_used(slot);
          float z[G];
#pragma unroll
          for (int h = 0; h < G; ++h) z[h] = zown[t][h];
          if (slot >= 0 && valid && !whole) {
#pragma unroll
            for (int h = 0; h < G; ++h)
              if (h < n_group) z_dec[(head0 + h) * n_slots + (d_lo + slot)] = z[h];
          }
#pragma unroll
          for (int h = 0; h < G; ++h) {
            const float w = scores_c ? exp2_of_whole_reference(z[h], ref[h]) : __builtin_amdgcn_exp2f(z[h] - ref[h]);
            const float p = valid ? w : 0.f;
            zown[t][h] = p;
            L[h] += p;
          }
        }
      };
      if (whole && b0 >= nb_p) take_weights(std::true_type{});  // these weights become scores, where tokens of equal keys tie
      else take_weights(std::false_type{});
      wave_lds_fence();

      // ---- pass 2: weighted values -----------------------------------------------------------------------
      if (LONG) {
        const int part = sum_part<S::kLanes>(lane);
#pragma unroll
        for (int j = 0; j < kOwnSums; ++j) {
          float a = alpha[j / E];
#pragma unroll
          for (int q = 1; q * kOwnSums < G * E; ++q) a = part == q ? alpha[(q * kOwnSums + j) / E] : a;
          sums[j] *= a;
        }
      }
      float o[G * E];
#pragma unroll
      for (int i = 0; i < G * E; ++i) o[i] = 0.f;
      auto use_rows = [&](int b, const u32x4 (&raw)[kBlockLoads]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kBlockLoads; ++u) {
          float vf[E];
          Widen<T>::get(raw[u], vf);
#pragma unroll
          for (int h = 0; h < G; ++h) {
            const float p = zown[(b - b0) / kWaves * S::kBlock + u * kRowsPerLoad + grp][h];
#pragma unroll
            for (int e = 0; e < E; ++e) o[h * E + e] = fmaf(p, vf[e], o[h * E + e]);
          }
        }
      };
#pragma clang loop unroll(disable)
      for (blk = b0 + wave; blk + kWaves < b1; blk += 2 * kWaves) {  // (a way out in its middle would copy the sums)
        load_rows(blk + kWaves, vraw[1]);
        use_rows(blk, vraw[0]);
        load_rows(blk + 2 * kWaves, vraw[0]);
        use_rows(blk + kWaves, vraw[1]);
      }
      if (blk < b1) use_rows(blk, vraw[0]);
      // The slot taking the new token was free, so it came as zeros: its value row is appended, whatever weight the token
      // got, and added here.
      if (takes_new && grp == 0) {
        *reinterpret_cast<u32x4*>(vd0 + static_cast<size_t>(new_row) * kRow + v_off) = v_of_new;
        float vf[E];
        Widen<T>::get(v_of_new, vf);
#pragma unroll
        for (int h = 0; h < G; ++h) {
          const float p = zown[(new_blk - b0) / kWaves * S::kBlock + new_row % S::kBlock][h];
#pragma unroll
          for (int e = 0; e < E; ++e) o[h * E + e] = fmaf(p, vf[e], o[h * E + e]);
        }
      }
      sum_scatter<S::kLanes>(o);
#pragma unroll
      for (int j = 0; j < kOwnSums; ++j) sums[j] += o[j];
      if (!LONG || b1 == n_blk) break;
    }

  // Sums over the waves, each with a maximum of its own.
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float l = wave_sum(L[h]);
    if (lane == 0) { s_sum[wave][h] = l; s_max[wave][h] = M[h]; }
  }
  // of head h over all waves: maximum and sum of weights
  auto merged = [&](int h, float& m, float& l) __attribute__((always_inline)) {
    m = s_max[0][h];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, s_max[w][h]);
    l = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
      l = fmaf(s_sum[w][h], s_max[w][h] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(s_max[w][h] - m), l);
  };
  if (whole && n_blk > 0 && n_d > 0) {  // (no piece was taken where the pool is full)
    // the weights of the slots are those of the last piece: each wave's are scaled to the softmax and summed over the heads
    __syncthreads();
    float f[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float m, l;
      merged(h, m, l);
      // (NaN where no wave has a finite logit, as in the finish kernel)
      f[h] = (M[h] != -INFINITY ? __builtin_amdgcn_exp2f(M[h] - m) : 0.f) * (1.f / l);
    }
    for (int t = lane; t < kOwnRows; t += kWave) {
      const int slot = (b0 - nb_p + wave + t / S::kBlock * kWaves) * S::kBlock + t % S::kBlock;
      if (slot >= n_d) break;
      float score = 0.f;
#pragma unroll
      for (int h = 0; h < G; ++h)
        if (h < n_group) score = fmaf(zown[t][h], f[h], score);
      z_dec[plane * n_slots + slot] = score;
    }
  }
  wave_lds_fence();
  float* s_o = &zown[0][0];  // [G][D], behind the weights
  if (S::kLanes != 8 || (lane & 8) == 0) {
#pragma unroll
    for (int j = 0; j < kOwnSums; ++j) {
      const int i = kOwnSums * sum_part<S::kLanes>(lane) + j;
      s_o[i / E * D + lane % S::kLanes * E + i % E] = sums[j];
    }
  }
  __syncthreads();
  for (int idx = tid; idx < G * D; idx += kThreads) {
    const int h = idx / D, dd = idx % D;
    if (h >= n_group) continue;
    float m, l;
    merged(h, m, l);
    float acc = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
      acc = fmaf((&zbuf[w][0][0])[idx], s_max[w][h] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(s_max[w][h] - m), acc);
    if (whole) {
      part_o[(head0 + h) * D + dd] = n_blk > 0 ? acc * (1.f / l) : 0.f;
      continue;
    }
    const size_t r = (head0 + h) * n_splits + split;
    part_o[r * D + dd] = acc;
    if (dd == 0) part_ml[r] = make_float2(m, l);
  }
}

}  // namespace

// Slots whose K rows the ranges of nothing but slots request ahead of the slot map, a trip to memory earlier: where a
// launch is one round of workgroups they would end it.  Whole steps, waiting for the map and ahead of it: 16 sequences of
// 4096 rows and 1025 slots 65.0 and 63.9 us, 8 38.5 and 38.0, 5 of 3414 and 1707 33.3 and 32.5, half full 30.8 and 29.8; in
// ranges of about a block per wave 4 of 700 and 501 17.7 and 17.1, 8 of 1000 and 2001, half full, 27.0 and 26.1, a tenth
// full 26.4 and 25.7.  Rows of free slots are fetched for nothing that way, so no more than can be in use are requested: a new token
// takes the lowest free slot, so a pool that is used from step 0 on is empty behind slot `step`, and behind slot `budget`
// (with all slots requested, a tenth full: 16 of 2561 and 2560, head_dim 64, 31.4 and 30.6 like this, 5 of 3414 and 1707, fp32 of
// head_dim 64, 25.5 and 24.1).  In more than one round other workgroups cover the trip (64 of 2000 and 1001, head_dim 64, half
// full, 77.3 ahead of the map and 76.3 behind it).
static int ahead_of_map(const DecodeDims& d, int row_bytes) {
  const long workgroups = static_cast<long>(d.n_splits) * d.H_kv * d.S;
  if (workgroups > decode_resident(d.G, row_bytes)) return 0;
  return min(d.n_slots - 1, min(d.step, d.budget)) + 1;
}

template <typename T, int D>
static hipError_t launch_partial(const DecodeDims& d, const shotkv_decode_state& st, const void* q_new,
                                 const void* k_new, const void* v_new, float* out, const DecodeWorkspace& w,
                                 hipStream_t s) {
  const int n_splits = d.whole ? 1 : d.n_splits, split_tokens = d.whole ? d.cap + d.n_slots : d.split_tokens;
  const dim3 grid(n_splits, d.H_kv, d.S), block(kThreads);
  const float c = d.sm_scale * kLog2e;
  const int ahead_slots = ahead_of_map(d, D * static_cast<int>(sizeof(T)));
  KernelTimer timer(d.timing, kKernelDecodePartial, s);
#define SHOTKV_LAUNCH_DEC(GG)                                                                           \
  auto* kernel = split_tokens > kMaxRange || d.whole ? decode_partial_kernel<T, D, GG, true>            \
                                                     : decode_partial_kernel<T, D, GG, false>;          \
  hipLaunchKernelGGL(kernel, grid, block, 0, s,                                                         \
                     static_cast<const char*>(st.k_prefill), static_cast<const char*>(st.v_prefill),    \
                     st.prefill_count, static_cast<char*>(st.k_dec), static_cast<char*>(st.v_dec),      \
                     st.slot_pos, d.cap, d.n_slots, d.H, d.H_kv, d.G, n_splits, split_tokens, ahead_slots, c, \
                     static_cast<const char*>(q_new), static_cast<const char*>(k_new),                  \
                     static_cast<const char*>(v_new), w.part_ml, d.whole ? out : w.part_o, w.z_dec, w.new_slot, d.whole)
  switch (padded_group(d.G)) {  // the kernel is instantiated for power-of-two groups and skips the padding
    case 1: { SHOTKV_LAUNCH_DEC(1); break; }
    case 2: { SHOTKV_LAUNCH_DEC(2); break; }
    case 4: { SHOTKV_LAUNCH_DEC(4); break; }
    case 8: { SHOTKV_LAUNCH_DEC(8); break; }
    default: return hipErrorInvalidValue;
  }
#undef SHOTKV_LAUNCH_DEC
  return hipGetLastError();
}

hipError_t launch_decode_partial(const DecodeDims& d, const shotkv_decode_state& st, const void* q_new,
                                 const void* k_new, const void* v_new, float* out, const DecodeWorkspace& w,
                                 hipStream_t s) {
  if (d.dtype == SHOTKV_BF16) {
    if (d.D == 128) return launch_partial<bf16_t, 128>(d, st, q_new, k_new, v_new, out, w, s);
    if (d.D == 64) return launch_partial<bf16_t, 64>(d, st, q_new, k_new, v_new, out, w, s);
  } else {
    if (d.D == 128) return launch_partial<float, 128>(d, st, q_new, k_new, v_new, out, w, s);
    if (d.D == 64) return launch_partial<float, 64>(d, st, q_new, k_new, v_new, out, w, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace shotkv
