// Shared device/host helpers for the ShotKV gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "shotkv.h"

namespace shotkv {

constexpr int kWave = 64;
constexpr float kLog2e = 1.4426950408889634f;

typedef uint16_t bf16_t;  // raw bf16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t x) {
  return __uint_as_float(static_cast<uint32_t>(x) << 16);
}
__device__ __forceinline__ float to_f32(bf16_t x) { return bf16_to_f32(x); }
__device__ __forceinline__ float to_f32(float x) { return x; }

// Value of lane (own lane ^ MASK), MASK a power of two below 64, without a trip through the LDS pipe:
// data-parallel-primitive moves inside a row of 16 lanes (1, 2: quad permutations; 4: the mirror of 8
// lanes followed by the mirror of 4; 8: a rotation of the row by 8), row swaps for 16 and half swaps for 32.
template <int MASK>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  static_assert(MASK == 1 || MASK == 2 || MASK == 4 || MASK == 8 || MASK == 16 || MASK == 32, "one lane bit");
  if constexpr (MASK == 1) {
    return __builtin_amdgcn_update_dpp(0u, v, 0xB1, 0xf, 0xf, false);   // quad_perm [1,0,3,2]
  } else if constexpr (MASK == 2) {
    return __builtin_amdgcn_update_dpp(0u, v, 0x4E, 0xf, 0xf, false);   // quad_perm [2,3,0,1]
  } else if constexpr (MASK == 4) {
    const uint32_t m = __builtin_amdgcn_update_dpp(0u, v, 0x141, 0xf, 0xf, false);  // row_half_mirror: lane ^ 7
    return __builtin_amdgcn_update_dpp(0u, m, 0x1B, 0xf, 0xf, false);               // quad_perm [3,2,1,0]: ^ 3
  } else if constexpr (MASK == 8) {
    return __builtin_amdgcn_update_dpp(0u, v, 0x128, 0xf, 0xf, false);  // row_ror:8
  } else if constexpr (MASK == 16) {
    // first result: own even rows, the other operand's even rows in the odd rows; second: the odd rows
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (threadIdx.x & 16) ? r[0] : r[1];
  } else {
    // first result: the lower half in both halves; second: the upper half in both
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (threadIdx.x & 32) ? r[0] : r[1];
  }
}

// Reductions over the wave, widest exchange first; every lane gets the result.  Six exchanges through the LDS pipe one
// after the other take a quarter of a microsecond, these a third of that.
template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T v, Op op) {
  static_assert(sizeof(T) == 4, "32-bit values");
  v = op(v, __builtin_bit_cast(T, lane_xor<32>(__builtin_bit_cast(uint32_t, v))));
  v = op(v, __builtin_bit_cast(T, lane_xor<16>(__builtin_bit_cast(uint32_t, v))));
  v = op(v, __builtin_bit_cast(T, lane_xor<8>(__builtin_bit_cast(uint32_t, v))));
  v = op(v, __builtin_bit_cast(T, lane_xor<4>(__builtin_bit_cast(uint32_t, v))));
  v = op(v, __builtin_bit_cast(T, lane_xor<2>(__builtin_bit_cast(uint32_t, v))));
  return op(v, __builtin_bit_cast(T, lane_xor<1>(__builtin_bit_cast(uint32_t, v))));
}
template <typename T>
__device__ __forceinline__ T wave_max(T v) {
  return wave_reduce(v, [](T a, T b) { return max(a, b); });
}
template <typename T>
__device__ __forceinline__ T wave_min(T v) {
  return wave_reduce(v, [](T a, T b) { return min(a, b); });
}
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
  return wave_reduce(v, [](T a, T b) { return a + b; });
}

// Combining a value with the one held 32 (or 16) lanes away without a trip through the LDS pipe: the
// half swap returns the lower half of the wave in both halves of its first result and the upper half in
// both halves of the second, the row swap does the same for each pair of 16-lane rows.
__device__ __forceinline__ float sum_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float max_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// The larger of two numbers in one instruction: fmaxf first quiets every operand of unknown origin by an instruction of its
// own.  Of a NaN and a number the number, of two NaNs infinity: only where a NaN makes everything that the maximum is used
// for NaN (a softmax reference that is carried on to keys without one takes fmaxf).
__device__ __forceinline__ float max_of_two(float a, float b) {
  float top = INFINITY;
  asm("" : "+s"(top));  // (a known constant would make it fmaxf again)
  return __builtin_amdgcn_fmed3f(a, b, top);
}
__device__ __forceinline__ float sum_across_row_pairs(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// reference + log2(sum), sum > 0.  The hardware logarithm errs low by a part of its result's last place, which for a sum
// of hundreds is 2^-20: only the mantissa goes through it, the exponent is exact.
__device__ __forceinline__ float add_log2(float reference, float sum) {
  return reference + static_cast<float>(__builtin_amdgcn_frexp_expf(sum)) +
         __builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(sum));
}

__host__ __device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Segments and chunks.  A problem's key axis is cut into segments - 0 the tokens before the first shot, s = 1..n
// shot s - 1, n + 1 the tokens after the last shot - and into slices of group_keys keys.  A chunk is the part of
// one segment that lies in one slice, so a chunk's softmax statistic belongs to one shot (or to the always-kept
// region) and to one score workgroup.  Its number is slice + segment: along the key axis every cut raises one of
// the two, so the numbers grow, no table of chunks is needed, and the chunks of one segment are consecutive
// (from first key / group_keys + s to last key / group_keys + s).  Numbers that no chunk has hold garbage.
__host__ __device__ __forceinline__ int max_chunks(int n_groups, int n_shots) { return n_groups + n_shots + 1; }

// ---- optional per-kernel timing (host) -----------------------------------------------------------

enum KernelKind {
  kKernelPlan = 0, kKernelScore, kKernelRowStats, kKernelChunkMass, kKernelReduceSelect, kKernelCompact,
  kKernelDecodePartial, kKernelDecodeFinish, kKernelPackVt, kKernelAttention, kKernelKinds
};
static_assert(kKernelKinds == SHOTKV_KERNEL_KINDS, "kernel kinds");

// Brackets one kernel launch with the caller's HIP events for that kind, if the caller passed any.  A kind whose work
// another kernel does is bracketed around nothing, so that kernel's time is counted under one kind only.
class KernelTimer {
 public:
  KernelTimer(void* const* events, KernelKind kind, hipStream_t stream)
      : stop_(events ? static_cast<hipEvent_t>(events[2 * kind + 1]) : nullptr), stream_(stream) {
    if (events) (void)hipEventRecord(static_cast<hipEvent_t>(events[2 * kind]), stream);
  }
  ~KernelTimer() {
    if (stop_) (void)hipEventRecord(stop_, stream_);
  }
  KernelTimer(const KernelTimer&) = delete;
  KernelTimer& operator=(const KernelTimer&) = delete;

 private:
  hipEvent_t stop_;
  hipStream_t stream_;
};

// ---- workspace carving (host) -------------------------------------------------------------------

struct PrefillWorkspace {
  // softmax partial per (problem, chunk, kv head, row): log2 of the chunk's sum of exponentials
  // (-inf for a row that sees none of the chunk's keys)
  float*   partial;       // [P][H_kv][maxC][R]
  // the same statistic over all chunks of a slice, which is what the row denominators are built from; the fused
  // attention kernel writes the denominator itself, as the statistic of a single slice
  float*   group_stat;    // [P][H_kv][n_groups][R]
  float*   chunk_mass;    // [P][maxC][H_kv]
  float*   scores;        // [P][n_shots]
  void*    vt;            // fused attention path only: V packed into 32-key blocks [P][H_kv][blocks][D][32], fp16
  uint32_t* v_absmax;     // fused attention path only: [P][H_kv] largest finite |v| of the plane, as bf16 bits
  uint32_t* v_share_max;  // fused attention path only: [P][H_kv][kVShares] the same of every share of the plane
  int32_t  max_c;
  int32_t  group_keys;    // keys per slice of the key axis, a power of two
  int32_t  n_groups;      // ceil(n_tokens / group_keys)
  size_t   bytes;
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr int kVShares = 128;        // shares of a V plane whose maxima are taken separately (fused attention path)
constexpr int kOneSlice = 1 << 30;   // group_keys where the whole key axis is one slice

int score_group_keys(int P, int H_kv, int row_blocks, int n_tokens, int n_shots);  // keys per workgroup of the score kernel

inline PrefillWorkspace carve_prefill(void* base, int P, int H_kv, int R, int n_tokens, int n_shots,
                                      int group_keys, size_t vt_bytes = 0) {
  PrefillWorkspace w{};
  w.group_keys = group_keys;
  w.n_groups = (n_tokens - 1) / group_keys + 1;
  w.max_c = max_chunks(w.n_groups, n_shots);
  size_t off = 0;
  char* b = static_cast<char*>(base);
  auto take = [&](size_t bytes) {
    char* p = b ? b + off : nullptr;
    off = align_up(off + bytes, 256);
    return p;
  };
  const size_t P_ = P, C = w.max_c, S = n_shots;
  w.partial = reinterpret_cast<float*>(take(P_ * H_kv * C * R * 4));
  w.group_stat = reinterpret_cast<float*>(take(P_ * H_kv * w.n_groups * R * 4));
  w.chunk_mass = reinterpret_cast<float*>(take(P_ * C * H_kv * 4));
  w.scores = reinterpret_cast<float*>(take(P_ * S * 4 + 4));
  w.vt = vt_bytes ? take(vt_bytes) : nullptr;
  w.v_absmax = vt_bytes ? reinterpret_cast<uint32_t*>(take(P_ * H_kv * 4)) : nullptr;
  w.v_share_max = vt_bytes ? reinterpret_cast<uint32_t*>(take(P_ * H_kv * kVShares * 4)) : nullptr;
  w.bytes = off;
  return w;
}

// ---- launchers implemented in the kernel files --------------------------------------------------

struct PrefillDims {
  int P, n_tokens, n_shots, H, H_kv, G, D, W;
  int R;       // row stride of the per-row workspace arrays: G * W, padded to the score kernel's blocks of 32 rows
  int R_rows;  // G * W query rows per KV head that really exist
  int dtype;
  float sm_scale;
  int select_mode;
  int share;  // consecutive problems that read one row of shot_offsets / budget_tokens
  void* const* timing;  // the caller's timing events, or null
};

hipError_t launch_score_partials(const PrefillDims& d, const void* q_obs, const void* k,
                                 const int32_t* shot_offsets, const PrefillWorkspace& w, hipStream_t s);
// Row denominators from the slices' statistics and, with them, every chunk's attention mass.  n_valid: rows of
// the R-row arrays that are written (the rest carries no weight).
hipError_t launch_chunk_mass(const PrefillDims& d, int n_valid, const PrefillWorkspace& w, hipStream_t s);
// Shot scores from the chunk masses (with_mass), the selection and copy plan (with_select), or both in
// one launch.  with_mass writes shot_scores; otherwise shot_scores is read.
hipError_t launch_reduce_select(const PrefillDims& d, bool with_mass, bool with_select, float* shot_scores,
                                const int32_t* shot_offsets, const int32_t* budget_tokens, int cap,
                                int32_t* kept_count, uint8_t* shot_selected, int32_t* status,
                                int32_t* kept_positions, const PrefillWorkspace& w, hipStream_t s);
// The selection and copy plan with the copies, in one launch or two.
hipError_t launch_select_compact(const PrefillDims& d, bool with_mass, float* shot_scores, const int32_t* shot_offsets,
                                 const int32_t* budget_tokens, const void* k, const void* v, void* k_out, void* v_out,
                                 int cap, int32_t* kept_count, uint8_t* shot_selected, int32_t* status,
                                 int32_t* kept_positions, const PrefillWorkspace& w, hipStream_t s);
hipError_t launch_compact(const PrefillDims& d, const void* k, const void* v, void* k_out, void* v_out,
                          int cap, const int32_t* kept_positions, const int32_t* kept_count,
                          hipStream_t s);

int score_row_blocks(int dtype, int rows);  // blocks of 32 query rows the score kernel is instantiated for

// causal attention forward that also writes the window rows' softmax partials and row denominators
bool attention_supported(const PrefillDims& d);
int attention_key_blocks(int n_tokens);
hipError_t launch_pack_vt(const PrefillDims& d, const void* v, const PrefillWorkspace& w, hipStream_t s);
hipError_t launch_attention_scores(const PrefillDims& d, const void* q, const void* k, const void* vt,
                                   const int32_t* shot_offsets, float* attn_out, const PrefillWorkspace& w, hipStream_t s);

struct DecodeDims {
  int S, H, H_kv, G, D, dtype, cap, n_slots, budget, step, n_splits, split_tokens;
  bool whole;  // one workgroup per sequence and KV head: n_splits and split_tokens only size the workspace
  float sm_scale;
  void* const* timing;  // the caller's timing events, or null
};

struct DecodeWorkspace {
  float2* part_ml;   // [S][H][n_splits] (max in log2 domain, sum)
  float*  part_o;    // [S][H][n_splits][D]
  // [S][H][n_slots] scaled logits (log2 domain) of the occupied decode slots; where one workgroup takes all of a
  // (sequence, KV head), [S][H_kv][n_slots] their weights summed over its query heads
  float*  z_dec;
  int32_t* new_slot;  // [S] slot chosen for the new token this step, -1 if the pool is full
  size_t  bytes;
};

inline DecodeWorkspace carve_decode(void* base, int S, int H, int H_kv, int D, int n_slots,
                                    int n_splits) {
  DecodeWorkspace w{};
  size_t off = 0;
  char* b = static_cast<char*>(base);
  auto take = [&](size_t bytes) {
    char* p = b ? b + off : nullptr;
    off = align_up(off + bytes, 256);
    return p;
  };
  const size_t S_ = S;
  w.part_ml = reinterpret_cast<float2*>(take(S_ * H * n_splits * 8));
  w.part_o = reinterpret_cast<float*>(take(S_ * H * n_splits * D * 4));
  w.z_dec = reinterpret_cast<float*>(take(S_ * H * n_slots * 4));
  w.new_slot = reinterpret_cast<int32_t*>(take(S_ * 4));
  w.bytes = off;
  return w;
}

// Tokens a decode workgroup can hold logits for in LDS at a time.
#ifndef SHOTKV_DEC_MAX_RANGE
#define SHOTKV_DEC_MAX_RANGE 1024
#endif
constexpr int kDecodeMaxRange = SHOTKV_DEC_MAX_RANGE;
constexpr int kDecodeMaxSplits = 1024;  // token ranges per (sequence, KV head) the finish kernel can merge

// query heads per KV head rounded up to 1, 2, 4 or 8: what the decode kernels are instantiated for
inline int padded_group(int G) { return G <= 1 ? 1 : G <= 2 ? 2 : G <= 4 ? 4 : G <= 8 ? 8 : 0; }

int decode_resident(int G, int row_bytes);  // workgroups of the decode kernel that the chip holds at once
int decode_splits(int S, int H_kv, int G, int row_bytes, int total_tokens);
// Slots whose map, and tokens whose logits, a decode workgroup of four waves holds in LDS: the blocks of rows that a wave
// takes at a time are dealt to the waves in turn.
constexpr int kDecodeBlockBytes = 4096;
constexpr int decode_map_rows(int row_bytes) {
  const int block = kDecodeBlockBytes / row_bytes;
  return (kDecodeMaxRange / block + 1 + 3) / 4 * 4 * block;
}
bool decode_whole(const DecodeDims& d, int row_bytes);
hipError_t launch_decode_partial(const DecodeDims& d, const shotkv_decode_state& st, const void* q_new,
                                 const void* k_new, const void* v_new, float* out, const DecodeWorkspace& w,
                                 hipStream_t s);
hipError_t launch_decode_finish(const DecodeDims& d, const shotkv_decode_state& st, float* out,
                                float* token_scores, int32_t* evicted_pos, int32_t* status,
                                const DecodeWorkspace& w, hipStream_t s);

}  // namespace shotkv
