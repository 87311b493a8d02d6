// Split-KV decode attention with the logits on the matrix cores
// (Section 5.1, Eq. 7 and 9: attention of the current query over prefill rows and decode slots).
//
// A workgroup owns one token range of one (sequence, KV head) and makes two passes over it, in pieces of at
// most kMaxRange tokens:
//   1. K pass: the logits of 4 or 8 tokens per matrix step, with the head dimension cut into pieces that
//      sit in different operand rows/columns, so that the A operands are whole K rows fetched straight
//      from global memory with coalesced 16-byte loads (RowShape).  The scaled logits go to LDS, their
//      maximum stays in registers.
//   between: weights 2^(z - max) by all threads, tokens along the lanes; decode-slot logits are also written
//      out for the retention score (Eq. 7).  The first V rows are already on their way: they are requested
//      between the loads of a wave's last K block and its use.
//   2. V pass: RowShape::kLanes lanes stream one V row each (16 bytes per lane) and accumulate weight * V with
//      the weights read from LDS, the next batch of rows in flight while one is used.  No rescaling is
//      needed because the maximum is already known.
// Bound by the stream of K and V rows: 32 query / 8 KV heads, head_dim 128 bf16, 512 caches of ~5000 rows 1.79 ms
// = 5.9 TB/s, 16 caches 58 us.  Before the rows of 64-dimensional heads and of fp32 caches took this form they
// were scored and summed by one-pass vector arithmetic: 32 caches of 2001 + 512 rows, head_dim 64, 57 us then,
// 33 us now; 8 caches of 2000 + 500 fp32 rows 57 -> 38 us a step.  Requesting the first V rows ahead of the
// weights is worth 4 us of 74 at 16 caches.
// Compared with a one-pass online softmax this moves the dot products off the vector ALU, removes the
// cross-lane reductions per token and the per-token rescale of the output accumulators.
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

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kMaxRange = kDecodeMaxRange;  // tokens whose logits the LDS buffer holds at a time
#ifndef SHOTKV_DEC_V_UNROLL
#define SHOTKV_DEC_V_UNROLL 4
#endif
constexpr int kVUnroll = SHOTKV_DEC_V_UNROLL;  // V rows a lane group has in flight

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
  static constexpr int kBlock = 8 * 1024 / ROW_BYTES;               // tokens a wave takes at a time (8 loads)
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

template <typename T, int D, int G, bool PIECES>
__global__ __launch_bounds__(kThreads, PIECES ? 2 : G == 8 ? 3 : 4) void decode_partial_kernel(
    const char* __restrict__ k_prefill, const char* __restrict__ v_prefill,
    const int32_t* __restrict__ prefill_count, char* __restrict__ k_dec, char* __restrict__ v_dec,
    const int32_t* __restrict__ slot_pos, int cap, int n_slots, int H, int H_kv, int n_group,
    int n_splits, int split_tokens, int ahead_slots, float scale_log2e, const char* __restrict__ q_new,
    const char* __restrict__ k_new, const char* __restrict__ v_new, float2* __restrict__ part_ml,
    float* __restrict__ part_o, float* __restrict__ z_dec, int32_t* __restrict__ new_slot_out) {
  constexpr int kRow = D * static_cast<int>(sizeof(T));  // bytes per row
  typedef RowShape<kRow> S;
  constexpr int E = Widen<T>::kElems;
  const int split = blockIdx.x, g = blockIdx.y, s = blockIdx.z;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);

  constexpr int kGroups = kThreads / S::kLanes;  // V rows the workgroup takes at a time
  constexpr int kBatchRows = kGroups * kVUnroll;
  static_assert(kBatchRows % S::kBlock == 0, "row counts padded to V batches are whole K blocks");
  // logits, then weights: the live prefill rows of a piece, then its slots, each padded to whole V batches
  __shared__ __attribute__((aligned(16))) float zbuf[kMaxRange + 2 * kBatchRows][G];
  __shared__ float s_max[kWaves][G];
  __shared__ float s_sum[kWaves][G];
  float (*s_o)[G][D] = reinterpret_cast<float (*)[G][D]>(&zbuf[0][0]);  // the waves' output sums, after the weights
  static_assert(kWaves * D <= kMaxRange, "output sums fit");
  __shared__ int s_red[2][kWaves];
  __shared__ int s_sp[kMaxRange];  // slot map of the decode slots of the piece

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

  // ---- K rows: block [row0, row0 + kBlock) of the `rows` rows that start at `base`.  Rows past the end re-read
  // the last one, so every address stays inside the plane; their logits are not used. --------------------------
  constexpr int kStepsPerBlock = 8 / S::kLoads;
  Vec kraw[8];
  auto load_block = [&](const char* base, int row0, int rows) __attribute__((always_inline)) {
    const char* at = base + static_cast<size_t>(row0) * kRow;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t r = min((i / S::kLoads) * S::kTokens + tau, rows - 1 - row0);
      kraw[i] = stream_load<Vec>(at + (r * kRow + (i % S::kLoads) * 256 + a_off));
    }
  };
  // A wave's first block is requested before the count of live rows has arrived (dead rows may hold anything).
  const int early_rows = min(range_end, cap) - range_begin;
  if (wave * S::kBlock < early_rows) load_block(kp + static_cast<size_t>(range_begin) * kRow, wave * S::kBlock, early_rows);
  // Only a range that reaches into the decode slots needs the slot that takes the new token, the lowest free
  // one, and the slot map of its (first) piece with the last occupied slot of it (a pool that is still filling
  // up is empty behind that); all come out of one round of loads.
  // A range of nothing but slots does not wait for the map with a wave's first K block if that begins among the first
  // ahead_slots slots (ahead_of_map); the whole block is requested, and a wave whose block was not requested asks for it
  // when the map is there.  A free slot may hold anything: its logits are not used, and the new token's row replaces what
  // its slot held.
  const bool early = !PIECES && range_begin >= cap &&
                     wave * S::kBlock < min(range_end - range_begin, ahead_slots - (range_begin - cap));
  int new_slot = n_slots, last_used = -1;
  if (range_end > cap) {
    constexpr int kBatch = 8;  // loads in flight per thread
    const int d_lo = max(range_begin - cap, 0), d_hi = min(range_begin + kMaxRange, range_end) - cap;
    int best = INT32_MAX;
    int pos[kBatch];
    auto load_map = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < kBatch; ++j) pos[j] = sp[min(i0 + j * kThreads, n_slots - 1)];
    };
    load_map(tid);
    if (early)  // behind the map, as loads return in order
      load_block(kd + static_cast<size_t>(range_begin - cap) * kRow, wave * S::kBlock, range_end - range_begin);
#pragma clang loop unroll(disable)
    for (int i0 = tid; i0 < n_slots && (best == INT32_MAX || i0 < d_hi); i0 += kBatch * kThreads) {
      if (i0 != tid) load_map(i0);
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const int i = min(i0 + j * kThreads, n_slots - 1);
        if (pos[j] < 0) best = min(best, i);
        if (i >= d_lo && i < d_hi) {
          s_sp[i - d_lo] = pos[j];
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

  const int grp = tid / S::kLanes, v_off = 16 * (tid % S::kLanes);
  float o[G][E], M[G], L[G];  // L: this thread's share of the sum of weights
#pragma unroll
  for (int h = 0; h < G; ++h) {
    M[h] = -INFINITY;
    L[h] = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) o[h][e] = 0.f;
  }

  // The range is taken in pieces that the logit buffer holds.  Only contexts of over a million tokens have more
  // than one (PIECES); a loop around the body costs the others registers for what the compiler moves out of it, and
  // this form has the register budget of two waves per SIMD for the same reason: 1.2 million rows, 32 query / 8 KV
  // heads, 1288 us with four (spills), 879 with three, 809 with two; 28 / 4 heads 969, 969 and 490; 16 / 4 at
  // head_dim 64 497, 282 and 240.
  const int n_pieces = PIECES ? ceil_div(range_end - range_begin, kMaxRange) : range_end > range_begin;
  if (new_slot >= 0)
#pragma clang loop unroll(disable)
    for (int piece = 0; piece < n_pieces; ++piece) {
      const bool first = !PIECES || piece == 0;
      const int t_begin = PIECES ? range_begin + piece * kMaxRange : range_begin;
      const int t_end = PIECES ? min(range_end, t_begin + kMaxRange) : range_end;
      const int n_p = max(min(t_end, pc) - t_begin, 0);         // live prefill rows of the piece
      const int d_lo = max(t_begin - cap, 0);                   // its decode slots: [d_lo, d_lo + n_d)
      const int n_d = max((first ? min(t_end - cap, last_used + 1) : t_end - cap) - d_lo, 0);
      const int new_row = new_slot >= d_lo && new_slot < d_lo + n_d ? new_slot - d_lo : -1;  // the new token's, if inside
      if (!first) {
        __syncthreads();  // the previous piece's weights and slot map are done with
        for (int i = tid; i < n_d; i += kThreads) s_sp[i] = sp[d_lo + i];
        __syncthreads();
      }
      const char* kp0 = kp + static_cast<size_t>(t_begin) * kRow;
      const char* vp0 = vp + static_cast<size_t>(t_begin) * kRow;
      char* kd0 = kd + static_cast<size_t>(d_lo) * kRow;
      char* vd0 = vd + static_cast<size_t>(d_lo) * kRow;
      auto slot_used = [&](int i) __attribute__((always_inline)) {
        return (i == new_row || s_sp[min(i, kMaxRange - 1)] >= 0) && i < n_d;
      };

      // ---- pass 1: logits --------------------------------------------------------------------------------
      const int z_d = ceil_div(n_p, kBatchRows) * kBatchRows;  // first entry of the slots in zbuf
      const int nb_p = ceil_div(n_p, S::kBlock), n_blk = nb_p + ceil_div(n_d, S::kBlock);
      float mx[kHeadSets];  // largest logit this lane has seen, of head col_head + kCols * m
#pragma unroll
      for (int m = 0; m < kHeadSets; ++m) mx[m] = -INFINITY;
      auto append = [&](int row0) __attribute__((always_inline)) {  // only this workgroup reads the slot this step
        if (new_row >= row0 && new_row < row0 + S::kBlock) {
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (row0 + (i / S::kLoads) * S::kTokens + tau == new_row) {
              kraw[i] = stream_load<Vec>(kn + (i % S::kLoads) * 256 + a_off);
              *reinterpret_cast<Vec*>(kd0 + static_cast<size_t>(new_row) * kRow + (i % S::kLoads) * 256 + a_off) =
                  kraw[i];
            }
        }
      };
      auto fetch = [&](int blk) __attribute__((always_inline)) {
        if (blk < nb_p) {
          load_block(kp0, blk * S::kBlock, n_p);
          return;
        }
        // A slot without a token is given an offset out of bounds, so it is zeros and costs no traffic, as in the V pass
        // (every other slot of 1025 free: 58.7 us a step for 16 caches of 4000 rows, 60.8 with all slots fetched).  A
        // block requested ahead of the map has its free slots fetched.
        const int row0 = (blk - nb_p) * S::kBlock;
        char* at = kd0 + static_cast<size_t>(row0) * kRow;
        const auto rows = __builtin_amdgcn_make_buffer_rsrc(at, 0, (n_d - row0) * kRow, kBufferFlags);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int r = (i / S::kLoads) * S::kTokens + tau;
          const bool used = s_sp[min(row0 + r, kMaxRange - 1)] >= 0;
          const int off = used ? r * kRow + (i % S::kLoads) * 256 + a_off : kOutOfBounds;
          kraw[i] = __builtin_bit_cast(Vec, __builtin_amdgcn_raw_buffer_load_b128(rows, off, 0, kNonTemporal));
        }
        append(row0);
      };
      // Logits of the block in kraw to zbuf[z0..]; counts(row, z): what the row at z0 + row adds to the maximum.
      auto multiply_block = [&](int z0, auto counts) __attribute__((always_inline)) {
#pragma unroll
        for (int st = 0; st < kStepsPerBlock; ++st) {
#pragma unroll
          for (int m = 0; m < kHeadSets; ++m) {
            const floatx4 acc = multiply_step<S::kLoads>(&kraw[st * S::kLoads], bq[m]);
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
              if (i16 < S::kCols && hq < G) zbuf[z0 + row][hq] = z;
            }
          }
        }
      };
      auto use_block = [&](int blk) __attribute__((always_inline)) {
        if (blk < nb_p) {
          // (a first block that was requested early holds dead rows behind the live ones)
          const int live = n_p - blk * S::kBlock;
          multiply_block(blk * S::kBlock, [&](int row, float z) { return row < live ? z : -INFINITY; });
        } else {
          const int row0 = (blk - nb_p) * S::kBlock;
          multiply_block(z_d + row0, [&](int row, float z) { return slot_used(row0 + row) ? z : -INFINITY; });
        }
      };
      int blk = wave;
      // the wave's first block: of the first piece it is there already if it lies among the live rows, or was requested
      // ahead of the slot map
      if (blk < n_blk) {
        if (first && early) append(blk * S::kBlock);
        else if (!(first && blk < nb_p)) fetch(blk);
      }
#pragma clang loop unroll(disable)
      for (; blk + kWaves < n_blk; blk += kWaves) {
        use_block(blk);
        fetch(blk + kWaves);
      }

      // V rows b * kBatchRows + u * kGroups + grp of the piece's live prefill rows (b < nv_p) or slots; for rows past
      // the end the buffer's bounds check returns zeros, at the price of a descriptor (a live row in their place, read
      // again, could be infinite: zero times that; 16 caches of 5121 rows 68.8 us that way, 69.4 like this, 70.8 with
      // the rows cleared after the load)
      const int nv_p = ceil_div(n_p, kBatchRows), n_v = nv_p + ceil_div(n_d, kBatchRows);
      u32x4 vraw[2][kVUnroll];
      auto load_rows = [&](int b, u32x4 (&raw)[kVUnroll]) __attribute__((always_inline)) {
        const bool in_p = b < nv_p;
        const int row0 = (in_p ? b : b - nv_p) * kBatchRows;
        char* at = const_cast<char*>(in_p ? vp0 : vd0) + static_cast<size_t>(row0) * kRow;
        const auto rows = __builtin_amdgcn_make_buffer_rsrc(at, 0, ((in_p ? n_p : n_d) - row0) * kRow, kBufferFlags);
#pragma unroll
        for (int u = 0; u < kVUnroll; ++u) {
          int off = (u * kGroups + grp) * kRow + v_off;
          if (!in_p && s_sp[min(row0 + u * kGroups + grp, kMaxRange - 1)] < 0) off = kOutOfBounds;
          raw[u] = __builtin_amdgcn_raw_buffer_load_b128(rows, off, 0, kNonTemporal);
        }
      };
      if (n_v > 0) load_rows(0, vraw[0]);  // in flight while the last logits and the weights are computed
      if (blk < n_blk) use_block(blk);

      // ---- between the passes: maximum, weights and their sum -----------------------------------------
#pragma unroll
      for (int m = 0; m < kHeadSets; ++m) {
        // lanes 16, 32 and 48 away hold other tokens of the same head (and so do, redundantly, the other pieces)
        const float w = max_across_halves(mx[m]);
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(w), __float_as_uint(w), false, false);
        const float wm = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
        const int hq = col_head + S::kCols * m;
        if (lane < S::kCols && hq < G) s_max[wave][hq] = wm;
      }
      __syncthreads();
      float ref[G];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float m_new = M[h];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) m_new = fmaxf(m_new, s_max[w][h]);
        if (!first) {  // a later piece: what the earlier ones gave moves to the new maximum
          const float alpha = M[h] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M[h] - m_new);
          L[h] *= alpha;
#pragma unroll
          for (int e = 0; e < E; ++e) o[h][e] *= alpha;
        }
        M[h] = m_new;
        ref[h] = m_new == -INFINITY ? 0.f : m_new;
      }
#pragma clang loop unroll(disable)
      for (int tt = tid; tt < n_v * kBatchRows; tt += kThreads) {
        const int slot = tt - z_d;
        const bool valid = slot < 0 ? tt < n_p : slot_used(slot);
        float z[G];
#pragma unroll
        for (int h = 0; h < G; ++h) z[h] = zbuf[tt][h];
        if (slot >= 0 && valid) {
#pragma unroll
          for (int h = 0; h < G; ++h)
            if (h < n_group) z_dec[(head0 + h) * n_slots + (d_lo + slot)] = z[h];
        }
#pragma unroll
        for (int h = 0; h < G; ++h) {
          const float p = valid ? __builtin_amdgcn_exp2f(z[h] - ref[h]) : 0.f;
          zbuf[tt][h] = p;
          L[h] += p;
        }
      }
      __syncthreads();

      // ---- pass 2: weighted values -----------------------------------------------------------------------
      auto use_rows = [&](int b, u32x4 (&raw)[kVUnroll]) __attribute__((always_inline)) {
        if (b >= nv_p) {
#pragma unroll
          for (int u = 0; u < kVUnroll; ++u) {
            const int row = (b - nv_p) * kBatchRows + u * kGroups + grp;
            // the slot taking the new token: its value row is appended whatever weight the token got
            if (row == new_row) {
              raw[u] = stream_load<u32x4>(vn + v_off);
              *reinterpret_cast<u32x4*>(vd0 + static_cast<size_t>(row) * kRow + v_off) = raw[u];
            }
          }
        }
#pragma unroll
        for (int u = 0; u < kVUnroll; ++u) {
          float vf[E];
          Widen<T>::get(raw[u], vf);
#pragma unroll
          for (int h = 0; h < G; ++h) {
            const float p = zbuf[b * kBatchRows + u * kGroups + grp][h];
#pragma unroll
            for (int e = 0; e < E; ++e) o[h][e] = fmaf(p, vf[e], o[h][e]);
          }
        }
      };
#pragma clang loop unroll(disable)
      for (int b = 0; b < n_v; b += 2) {
        if (b + 1 < n_v) load_rows(b + 1, vraw[1]);
        use_rows(b, vraw[0]);
        if (b + 1 >= n_v) break;
        if (b + 2 < n_v) load_rows(b + 2, vraw[0]);
        use_rows(b + 1, vraw[1]);
      }
      if (!PIECES) break;
    }

  // sum over the row groups of a wave, then over the waves
#pragma unroll
  for (int h = 0; h < G; ++h) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if constexpr (S::kLanes == 8) o[h][e] += row_rotate<8>(o[h][e]);
      if constexpr (S::kLanes <= 16) o[h][e] = sum_across_row_pairs(o[h][e]);
      o[h][e] = sum_across_halves(o[h][e]);
    }
    const float l = wave_sum(L[h]);
    if (lane == 0) s_sum[wave][h] = l;
  }
  __syncthreads();  // every wave is done with the weights
  if (lane < S::kLanes) {
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int e = 0; e < E; ++e) s_o[wave][h][lane * E + e] = o[h][e];
  }
  __syncthreads();
  for (int idx = tid; idx < G * D; idx += kThreads) {
    const int h = idx / D, dd = idx % D;
    if (h >= n_group) continue;
    float acc = 0.f, l = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      acc += s_o[w][h][dd];
      l += s_sum[w][h];
    }
    const size_t r = (head0 + h) * n_splits + split;
    part_o[r * D + dd] = acc;
    float m = M[0];
#pragma unroll
    for (int i = 1; i < G; ++i) m = i == h ? M[i] : m;
    if (dd == 0) part_ml[r] = make_float2(m, l);
  }
}

}  // namespace

// Slots whose K rows the ranges of nothing but slots request ahead of the slot map, a trip to memory earlier: where a
// launch is one round of workgroups they would end it (16 sequences of 4096 rows and 1025 slots 64.4 us a step waiting for
// the map and 63.5 ahead of it, 8 sequences 40.6 and 39.3, 16 of 2561 and 2560 74.0 and 71.6; 5 of 3414 and 1707, half
// full, 30.5 and 29.1).  Rows of free slots are fetched for nothing that way, so no more than can be in use are requested:
// a new token takes the lowest free slot, so a pool that is used from step 0 on is empty behind slot `step`, and behind
// slot `budget` (with all slots requested an empty pool of 4096 beside 256 rows took 26.8 us, 25.5 without; so it is 25.3).
// Ranges that a workgroup's waves take in little more than one block each have all their rows in flight at once and gain
// only while slots are few: 3 sequences in ranges of 160 rows 23.7 and 23.3 us with a tenth of slots, 28.5 and 28.4 with a
// third, 35.2 and 35.7 with two thirds; 8 of head_dim 64 in ranges of 196 rows 25.0 and 25.6 with two thirds.
static int ahead_of_map(const DecodeDims& d, int row_bytes) {
  const long workgroups = static_cast<long>(d.n_splits) * d.H_kv * d.S;
  if (workgroups > decode_resident(d.G, row_bytes)) return 0;
  if (d.split_tokens < 256 && d.cap / 2 < d.n_slots) return 0;
  return min(d.n_slots - 1, min(d.step, d.budget)) + 1;
}

template <typename T, int D>
static hipError_t launch_partial(const DecodeDims& d, const shotkv_decode_state& st, const void* q_new,
                                 const void* k_new, const void* v_new, const DecodeWorkspace& w, hipStream_t s) {
  const dim3 grid(d.n_splits, d.H_kv, d.S), block(kThreads);
  const float c = d.sm_scale * kLog2e;
  const int ahead_slots = ahead_of_map(d, D * static_cast<int>(sizeof(T)));
  KernelTimer timer(d.timing, kKernelDecodePartial, s);
#define SHOTKV_LAUNCH_DEC(GG)                                                                           \
  auto* kernel = d.split_tokens > kMaxRange ? decode_partial_kernel<T, D, GG, true>                     \
                                            : decode_partial_kernel<T, D, GG, false>;                   \
  hipLaunchKernelGGL(kernel, grid, block, 0, s,                                                         \
                     static_cast<const char*>(st.k_prefill), static_cast<const char*>(st.v_prefill),    \
                     st.prefill_count, static_cast<char*>(st.k_dec), static_cast<char*>(st.v_dec),      \
                     st.slot_pos, d.cap, d.n_slots, d.H, d.H_kv, d.G, d.n_splits, d.split_tokens, ahead_slots, c, \
                     static_cast<const char*>(q_new), static_cast<const char*>(k_new),                  \
                     static_cast<const char*>(v_new), w.part_ml, w.part_o, w.z_dec, w.new_slot)
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
                                 const void* k_new, const void* v_new, const DecodeWorkspace& w,
                                 hipStream_t s) {
  if (d.dtype == SHOTKV_BF16) {
    if (d.D == 128) return launch_partial<bf16_t, 128>(d, st, q_new, k_new, v_new, w, s);
    if (d.D == 64) return launch_partial<bf16_t, 64>(d, st, q_new, k_new, v_new, w, s);
  } else {
    if (d.D == 128) return launch_partial<float, 128>(d, st, q_new, k_new, v_new, w, s);
    if (d.D == 64) return launch_partial<float, 64>(d, st, q_new, k_new, v_new, w, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace shotkv
