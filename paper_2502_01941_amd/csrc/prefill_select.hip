// Per-shot scores from the chunk masses, whole-shot selection under the token budget and the copy plan
// for compaction (Section 5.1, Eq. 3-6; Algorithm 1 phase 1: score every shot, rank by score, keep
// shots in descending order while the budget holds).  One workgroup per problem does all of it:
//
//   scores    Score(s_i) = (sum of the masses of the shot's chunks) / k_i;
//   budget    prefix selection needs no ranking, only where in it the budget ends: up to 128 shots a group of lanes
//             per shot adds the lengths of all that rank no lower; above, the key of the shot at which the budget ends
//             is found a digit at a time from histograms of lengths (in LDS; integer sums, so their order is free);
//   ranking   first fit walks all shots in order: up to 128 shots a group of lanes per shot counts the ones above, more
//             are sorted: bitonic sort on one 64-bit key per shot (score descending, shot index
//             ascending): keys live in registers, partners less than 64 apart are exchanged between lanes without LDS
//             (DPP moves inside a row of 16, row and half swaps beyond), and for the larger strides the keys pass
//             through LDS into a transposed layout in which those strides are lane distances too - two LDS round trips
//             per merge level instead of one per compare-exchange step;
//   plan      sums of kept lengths in position order give every retained row's output slot; the segments that keep
//             tokens are numbered by the same pass, so that the original positions, written in ascending order, take a
//             group of lanes for each of these and none for the others;
//   copies    where there are few, by as many workgroups as there are CUs, each of which does all of the above for itself
//             (launch_select_compact); otherwise the positions go to the copying kernel.
//
// Bound by a chain of barriers and trips to memory in one workgroup.  Inside the kernel, sorting and walking the sums
// against this: 40 shots 2.1 + 1.8 us and 0.6, 80 shots 3.4 + 1.5 and 1, 600 units 7.8 + 1.7 and 3.3 (the sort of 400
// shots for first fit is 7.5); writing the positions of 600 units 4.0 and 1.9.  Whole call: 8192 tokens in 40 shots
// 29.5 -> 26.6 us, 16 x 16001 tokens of head_dim 64 in 80 shots 117.8 -> 113.5, 64 x 600 units 159.6 -> 150.8.  First fit,
// sorting against counting: 13 x 1424 tokens in 4 shots 36.6 -> 33.9, 60 problems of 109 shots 112.2 -> 109.7.
//
// The two halves can also run alone: scores only, or selection from caller-supplied scores.  All
// sums of floats run in a fixed order, so results are reproducible run to run.
#include "common.hpp"

#include <type_traits>

namespace shotkv {

namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;

// Inclusive sum over the lanes up to the own one, without a trip through the LDS pipe: shifts inside a row of 16 lanes,
// then the last lane of a row (of the lower half) to the rows behind it.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Exclusive sums over all threads of two values at once; total_a and total_b are the sums.  tmp: 2 * kSelWaves ints.
__device__ __forceinline__ void block_exclusive_scan(int& a, int& b, int& total_a, int& total_b, int* tmp) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int incl_a = wave_inclusive_scan(a), incl_b = wave_inclusive_scan(b);
  if (lane == kWave - 1) { tmp[wave] = incl_a; tmp[kSelWaves + wave] = incl_b; }
  __syncthreads();
  int before_a = 0, before_b = 0;
  total_a = total_b = 0;
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) {
    const int ta = tmp[w], tb = tmp[kSelWaves + w];
    if (w < wave) { before_a += ta; before_b += tb; }
    total_a += ta;
    total_b += tb;
  }
  a = before_a + incl_a - a;
  b = before_b + incl_b - b;
}

constexpr int kMaxPad = SHOTKV_MAX_SHOTS;            // keys sorted at most (a power of two)
constexpr int kKeySlots = kMaxPad + kMaxPad / 64;    // one pad slot per 64 keys: transposed reads hit all banks
static_assert((kMaxPad & (kMaxPad - 1)) == 0 && kMaxPad <= 4 * kSelThreads, "up to four keys per thread");
constexpr int kFewShots = kSelThreads / 8;           // shots that are ranked by counting, eight lanes or more to each
constexpr int kMinPad = 2 * kFewShots;               // keys sorted at least

// One key per shot whose descending order is the ranking: score descending, then index ascending.
// The float's bits are mapped to an unsigned integer with the same order (-0 ranks with +0); entry i
// of the padding (i >= n_shots) gets the smallest score word and therefore ranks after every shot.
__device__ __forceinline__ uint32_t score_word(float score) {
  uint32_t b = __float_as_uint(score);
  if ((b << 1) == 0u) b = 0u;
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ uint64_t rank_key(float score, int idx) {
  return (static_cast<uint64_t>(score_word(score)) << 32) | (0xFFFFFFFFu - static_cast<uint32_t>(idx));
}
__device__ __forceinline__ uint64_t padding_key(int idx) { return 0xFFFFFFFFu - static_cast<uint32_t>(idx); }

template <int MASK>
__device__ __forceinline__ uint64_t lane_xor64(uint64_t v) {
  const uint32_t lo = lane_xor<MASK>(static_cast<uint32_t>(v));
  const uint32_t hi = lane_xor<MASK>(static_cast<uint32_t>(v >> 32));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Sorts n_pad keys (a power of two, kMinPad <= n_pad <= E * 1024) into descending order.  Thread tid holds
// array elements tid + 1024 * j in k[j]; on return k[j] is the key of rank tid + 1024 * j.  All 1024
// threads must call it (barriers); threads whose elements lie past n_pad carry dummies.
// Layouts: "natural" - element t = tid + 1024 j is array index t; "transposed" - it is array index
// ((t mod 2^hb) << 6) | (t >> hb) with hb = log2(n_pad) - 6, which puts index bits 6.. on the low lane
// bits.  keys[] holds kKeySlots entries; array index a lives in slot a + a/64.  With n_pad <= 2048 two
// alternating buffers make one barrier per layout change enough; 4096 keys need a second one.
template <int E>
__device__ void sort_keys_descending(uint64_t (&k)[E], int n_pad, uint64_t* keys) {
  const int tid = threadIdx.x;
  const int hb = (31 - __clz(n_pad)) - 6;
  const int low_mask = (1 << hb) - 1;
  const int second = n_pad <= kMaxPad / 2 ? kKeySlots / 2 : 0;
  int buf = 0;
  auto natural = [&](int j) { return tid + kSelThreads * j; };
  auto transposed = [&](int j) {
    const int t = tid + kSelThreads * j;
    return ((t & low_mask) << 6) | (t >> hb);
  };
  auto slot = [](int a) { return a + (a >> 6); };
  // one compare-exchange step with the partner LANE_MASK lanes away: array distance LANE_MASK in the
  // natural layout, 64 * LANE_MASK in the transposed one
  auto stage = [&](int size, auto lane_mask_c, bool in_transposed) {
    constexpr int LANE_MASK = decltype(lane_mask_c)::value;
    const int stride = in_transposed ? LANE_MASK << 6 : LANE_MASK;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int a = in_transposed ? transposed(j) : natural(j);
      const uint64_t other = lane_xor64<LANE_MASK>(k[j]);
      const bool want_max = ((a & size) == 0) == ((a & stride) == 0);
      const bool take = want_max ? other > k[j] : other < k[j];
      k[j] = take ? other : k[j];
    }
  };
  // the steps of one merge level whose partners are at most `top` lanes away, widest first
  auto lane_stages = [&](int size, int top, bool in_transposed) {
    if (top >= 32) stage(size, std::integral_constant<int, 32>{}, in_transposed);
    if (top >= 16) stage(size, std::integral_constant<int, 16>{}, in_transposed);
    if (top >= 8) stage(size, std::integral_constant<int, 8>{}, in_transposed);
    if (top >= 4) stage(size, std::integral_constant<int, 4>{}, in_transposed);
    if (top >= 2) stage(size, std::integral_constant<int, 2>{}, in_transposed);
    stage(size, std::integral_constant<int, 1>{}, in_transposed);
  };
  auto relayout = [&](bool to_transposed) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int t = natural(j);
      if (t < n_pad) keys[buf + slot(to_transposed ? t : transposed(j))] = k[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int t = natural(j);
      if (t < n_pad) k[j] = keys[buf + slot(to_transposed ? transposed(j) : t)];
    }
    if (second) buf ^= second;
    else __syncthreads();
  };
  for (int size = 2; size <= n_pad; size <<= 1) {
    if (size > kWave) {
      relayout(true);
      lane_stages(size, size >> 7, true);   // array distances size/2 .. 64
      relayout(false);
    }
    lane_stages(size, min(size >> 1, kWave / 2), false);
  }
}

// First fit over the ranking by one wave, 64 ranks at a time: len[r] and shot[r] of rank r, keep[shot] = 1 where it
// still fits.  A shot longer than what is left can never fit again, so only the others are candidates; the ones
// ahead of the first candidate that overflows the running sum are kept together, that one is skipped, and the
// rest go on with what is left.  A walk by one thread reads two words of LDS per rank one
// after the other: this kernel took 43 us for 8 problems of 400 shots with it, 23 us with this one.
__device__ void first_fit_walk(const int* len, const uint16_t* shot, int n, int left, uint8_t* keep) {
  const int lane = threadIdx.x;
  for (int r0 = 0; r0 < n; r0 += kWave) {
    const int r = r0 + lane;
    const int my_len = r < n ? len[r] : 0;
    bool open = r < n && my_len <= left, taken = false;
    while (__builtin_amdgcn_ballot_w64(open) != 0) {
      const int incl = wave_inclusive_scan(open ? my_len : 0);
      const uint64_t over = __builtin_amdgcn_ballot_w64(open && incl > left);
      const int first = over ? __builtin_ctzll(over) : kWave;  // the first candidate that does not fit
      if (open && lane < first) taken = true;
      const int used = first > 0 ? __builtin_amdgcn_readlane(incl, first - 1) : 0;
      left -= used;
      open = open && lane > first && my_len <= left;
    }
    if (taken) keep[shot[r]] = 1;
  }
}

// Whether each of a thread's shots (threadIdx.x + 1024 * j) is among the first of the ranking that fit into `left` tokens
// together.  No ranking is needed for that, only the shot at which the budget ends: its key - score descending, then
// index ascending, 44 bits - is found a digit of eight bits at a time, from a histogram of the lengths over the digit of
// the keys that share the digits before.  A digit that one key has ends the search.  Keys share the first digits - sign,
// exponent and leading bits of the mantissa - the more of them the closer the scores lie: two or three rounds where they
// are spread over several powers of two, three or four within 10 % or 1 % of each other, four or five within 0.1 %, six
// where they are equal (the last two are the index), each 0.6 - 1 us and more where all keys add to one word.  Selection
// and copies of shots of 8 tokens, one problem, by the sort and by digits: 200 shots 12.8 us and 8.8 spread, 9.8 within
// 1 %, 10.7 within 0.1 %, 12.5 equal; 600 17.1 and 9.4, 11.6, 11.7, 14.0; 4096 55 and 17.8, 23, 24.5, 34.2; 64 problems of
// 600 29.9 and 23.5, 25.1, 25.7, 27.0.
// hist: kDigits * 256 words, cleared.  All threads call it, after a barrier behind the clearing.
constexpr int kDigits = 6;
__device__ __forceinline__ void keep_prefix(const float (&score)[kMaxPad / kSelThreads],
                                            const int (&len)[kMaxPad / kSelThreads], int n, int left, uint64_t* hist,
                                            bool (&keep)[kMaxPad / kSelThreads]) {
  constexpr int kPer = kMaxPad / kSelThreads;
  constexpr int kCount = 40;  // a word is count << 40 | tokens
  static_assert(kMaxPad <= 1 << 12, "indexes of 12 bits");
  const int tid = threadIdx.x, lane = tid % kWave;
  uint64_t key[kPer];
  bool open[kPer];  // shares the digits so far with the shot at which the budget ends
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = tid + kSelThreads * j;
    key[j] = static_cast<uint64_t>(score_word(score[j])) << 12 | static_cast<uint32_t>(kMaxPad - 1 - i);
    open[j] = i < n;
    keep[j] = false;
  }
#pragma clang loop unroll(disable)
  for (int digit = 0; digit < kDigits; ++digit, hist += 256) {
    const int shift = max(36 - 8 * digit, 0);
    int d[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      d[j] = static_cast<int>(key[j] >> shift) & (digit == kDigits - 1 ? 15 : 255);
      if (open[j])
        atomicAdd(reinterpret_cast<unsigned long long*>(&hist[d[j]]), 1ull << kCount | static_cast<unsigned>(len[j]));
    }
    __syncthreads();
    // every wave looks through all digits, highest first, four to a lane
    uint64_t word[4];
    int tokens = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      word[q] = hist[255 - 4 * lane - q];
      tokens += static_cast<int>(word[q]);
    }
    int before = wave_inclusive_scan(tokens) - tokens;
    const uint64_t over = __builtin_amdgcn_ballot_w64(before + tokens > left);
    int at = -1, count = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = static_cast<int>(word[q]);
      if (at < 0 && before + t > left) {
        at = 255 - 4 * lane - q;
        count = static_cast<int>(word[q] >> kCount);
      }
      if (at < 0) before += t;
    }
    const int first = over ? __builtin_ctzll(over) : 0;
    at = over ? __builtin_amdgcn_readlane(at, first) : -1;  // all fit: every digit is above
    left -= over ? __builtin_amdgcn_readlane(before, first) : 0;
    count = over ? __builtin_amdgcn_readlane(count, first) : 1;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      keep[j] |= open[j] && d[j] > at;
      open[j] = open[j] && d[j] == at;
    }
    if (count == 1) break;  // the shot at which the budget ends, or none
  }
}

// The same for few shots, without the rounds: a group of lanes per shot adds the lengths of all that rank no lower, or, for
// first fit, counts them.  word_add: n words, score word << 32 | what the shot adds, behind a barrier.  lanes: per shot, 8
// or 16.  Returned to all of the group.
__device__ __forceinline__ int sum_of_no_lower(const uint64_t* word_add, int n, int i, int part, int lanes) {
  const uint32_t own = i < n ? static_cast<uint32_t>(word_add[i] >> 32) : 0u;
  int sum = 0;
#pragma unroll 4
  for (int j = part; j < n; j += lanes) {
    const uint64_t x = word_add[j];
    const uint32_t word = static_cast<uint32_t>(x >> 32);
    sum += (word > own) | ((word == own) & (j <= i)) ? static_cast<int>(x) : 0;
  }
  sum += static_cast<int>(lane_xor<1>(static_cast<uint32_t>(sum)));
  sum += static_cast<int>(lane_xor<2>(static_cast<uint32_t>(sum)));
  sum += static_cast<int>(lane_xor<4>(static_cast<uint32_t>(sum)));
  if (lanes == 16) sum += static_cast<int>(lane_xor<8>(static_cast<uint32_t>(sum)));
  return sum;
}

// Sum of words[first], words[first + width], ... of n words: kBatch loads in flight, added up as a tree.
template <int kBatch, typename Load>
__device__ __forceinline__ float strided_sum(int n, int first, int width, Load word) {
  float sum = 0.f;
#pragma clang loop unroll(disable)
  for (int e0 = first; e0 < n; e0 += kBatch * width) {
    float x[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) x[j] = word(min(e0 + j * width, n - 1));
#pragma unroll
    for (int j = 0; j < kBatch; ++j) x[j] = e0 + j * width < n ? x[j] : 0.f;
#pragma unroll
    for (int o = kBatch / 2; o > 0; o >>= 1)
#pragma unroll
      for (int j = 0; j < o; ++j) x[j] += x[j + o];
    sum += x[0];
  }
  return sum;
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// The caches that a launch that copies as well reads and writes.
struct CopyArgs {
  const char* k;
  const char* v;
  char* k_out;
  char* v_out;
};

// ROW_BYTES: bytes of a cache row where the workgroups of a problem (blockIdx.x) also copy a share of its rows each, 0
// where they do not.  Each of them then makes the whole selection for itself; the first one writes it down.
template <bool MASS, bool SELECT, int ROW_BYTES>
__global__ __launch_bounds__(kSelThreads) void reduce_select_kernel(
    const float* __restrict__ chunk_mass, int max_c, int group_shift, int H_kv,
    float* __restrict__ shot_scores,
    const int32_t* __restrict__ shot_offsets, const int32_t* __restrict__ budget_tokens, int share,
    int n_shots, int n_tokens, int cap, int select_mode, int32_t* __restrict__ kept_count,
    uint8_t* __restrict__ shot_selected, int32_t* __restrict__ status,
    int32_t* __restrict__ kept_positions, CopyArgs copy) {
  const int p = blockIdx.y, tid = threadIdx.x;
  const bool writes = ROW_BYTES == 0 || blockIdx.x == 0;
  const int32_t* off_g = shot_offsets + static_cast<size_t>(p / share) * (n_shots + 1);
  float* scores = shot_scores + static_cast<size_t>(p) * n_shots;

  __shared__ int s_off[SHOTKV_MAX_SHOTS + 1];
  __shared__ uint64_t s_key[kKeySlots];       // histograms or the sort's exchange buffer, then (as ints) first rows
  __shared__ uint16_t s_idx[SHOTKV_MAX_SHOTS + 2];  // the ranking, then the segments that keep tokens
  __shared__ uint8_t s_keep[SHOTKV_MAX_SHOTS];
  __shared__ int s_tmp[2 * kSelWaves];
  __shared__ int s_flag;
  __shared__ float s_sum[kSelThreads / 2];    // mass of every shot, where a shot has more than one lane
  int* s_a = reinterpret_cast<int*>(s_key);   // SHOTKV_MAX_SHOTS + 3 ints
  static_assert(sizeof(uint64_t) * kKeySlots >= sizeof(int) * (SHOTKV_MAX_SHOTS + 3), "first rows fit");
  static_assert(kKeySlots >= kDigits * 256, "histograms fit");

  // ---- shot boundaries into LDS, validated: 0 <= off[0], strictly increasing, off[n] <= n_tokens --
  if (tid == 0) s_flag = 0;
  if (SELECT)
    for (int i = tid; i < kDigits * 256; i += kSelThreads) s_key[i] = 0;
  const int budget = SELECT ? budget_tokens[p / share] : 0;  // (requested with the boundaries)
  __syncthreads();
  int local_bad = 0;
  for (int i = tid; i <= n_shots; i += kSelThreads) {
    const int o = off_g[i];
    s_off[i] = o;
    if (o < 0 || o > n_tokens) local_bad = 1;
    if (i > 0 && o <= off_g[i - 1]) local_bad = 1;
  }
  if (local_bad) atomicOr(&s_flag, 1);
  __syncthreads();
  const bool bad = s_flag != 0;

  // ---- Eq. 3: one score per shot from the masses of its chunks ----------------------------------
  // Shot i is segment i + 1: its chunks' masses are consecutive, one word per KV head each.  A unit of thousands of
  // tokens is hundreds of words, which one thread would read one after the other; a group of lanes takes it, each with
  // at least eight words to add (fewer cost more in the exchange than they save: 8192 tokens in 40 shots, 14 words
  // each, 29.5 us with one lane and 30.3 with sixteen) and sixteen loads in flight, or four of 16 bytes where units are
  // many and short (whole call, 32768 tokens in 4000 units: 132 us, 143 with eight of 4 bytes).  Whole call, 32 query / 8 KV heads,
  // one thread per shot with one load at a time against this: 4000 tokens in 2 units 32.7 / 25.6 us, 8192 in 2
  // 38.9 / 31.5, 32768 in 4 57.9 / 47.2, 131072 in one 144 / 79.  The sums are also more exact than one long one.
  auto shot_sum = [&](int i, int first, int width) {
    const int lo = s_off[i], hi = s_off[i + 1];
    const int c0 = (lo >> group_shift) + i + 1, c1 = ((hi - 1) >> group_shift) + i + 1;
    const float* words = chunk_mass + (static_cast<size_t>(p) * max_c + c0) * H_kv;
    const int n = (c1 - c0 + 1) * H_kv;
    if (n_shots > kSelThreads / 2 && H_kv % 4 == 0) {  // one lane per unit, which has H_kv words per chunk
      const float4* quads = reinterpret_cast<const float4*>(words);
      return strided_sum<4>(n / 4, first, width, [&](int e) {
        const float4 x = quads[e];
        return (x.x + x.y) + (x.z + x.w);
      });
    }
    return strided_sum<16>(n, first, width, [&](int e) { return words[e]; });
  };
  int width = 1;
  if (MASS) {
    const int words = ((n_tokens >> group_shift) + n_shots) * H_kv;  // of all shots together
    while (width < kWave && 2 * width * n_shots <= kSelThreads && 16 * width * n_shots <= words) width <<= 1;
  }
  if (MASS && !bad && width > 1) {  // (the choice is the same for the whole workgroup)
    const int i = tid / width;
    float sum = i < n_shots ? shot_sum(i, tid % width, width) : 0.f;
    auto add = [&](auto mask_c) {
      constexpr int MASK = decltype(mask_c)::value;
      if (width > MASK) sum += __uint_as_float(lane_xor<MASK>(__float_as_uint(sum)));  // (width is uniform)
    };
    add(std::integral_constant<int, 32>{});
    add(std::integral_constant<int, 16>{});
    add(std::integral_constant<int, 8>{});
    add(std::integral_constant<int, 4>{});
    add(std::integral_constant<int, 2>{});
    add(std::integral_constant<int, 1>{});
    if (i < n_shots && tid % width == 0) s_sum[i] = sum;
    __syncthreads();
  }
  // thread tid takes shots tid, tid + 1024, ...: the layout the sort starts from
  constexpr int kMaxPerThread = kMaxPad / kSelThreads;
  float my_score[kMaxPerThread];
#pragma unroll
  for (int j = 0; j < kMaxPerThread; ++j) {
    const int i = tid + kSelThreads * j;
    my_score[j] = 0.f;
    if (i >= n_shots) continue;
    if (MASS) {
      if (!bad)
        my_score[j] = (width > 1 ? s_sum[i] : shot_sum(i, 0, 1)) / static_cast<float>(s_off[i + 1] - s_off[i]);
      if (writes) scores[i] = my_score[j];
    } else if (!bad) {
      my_score[j] = scores[i];
    }
  }
  if (!SELECT) {
    if (tid == 0) status[p] = bad ? SHOTKV_ST_BAD_OFFSETS : SHOTKV_ST_OK;
    return;
  }

  uint8_t* sel = shot_selected ? shot_selected + static_cast<size_t>(p) * n_shots : nullptr;
  int32_t* kept_pos = kept_positions + static_cast<size_t>(p) * cap;
  int st = bad ? SHOTKV_ST_BAD_OFFSETS : SHOTKV_ST_OK;
  int shot_budget = 0, n_prefix = 0, n_tail = 0;
  if (st == SHOTKV_ST_OK) {
    n_prefix = s_off[0];
    n_tail = n_tokens - s_off[n_shots];
    shot_budget = min(budget, cap) - n_prefix - n_tail;
    if (shot_budget < 0) st = SHOTKV_ST_BUDGET_TOO_SMALL;
  }
  if (st != SHOTKV_ST_OK) {
    if (!writes) return;
    if (tid == 0) { status[p] = st; kept_count[p] = 0; }
    if (sel) for (int i = tid; i < n_shots; i += kSelThreads) sel[i] = 0;
    return;
  }

  const bool prefix = select_mode == SHOTKV_SELECT_PREFIX;
  if (n_shots <= kFewShots) {
    // Rounds of the histogram cost 0.6 us each, this about as much in all: 40 shots 27.5 us a call with the histogram.
    if (tid < n_shots)
      s_key[tid] = static_cast<uint64_t>(score_word(my_score[0])) << 32 |
                   (prefix ? static_cast<uint32_t>(s_off[tid + 1] - s_off[tid]) : 1u);
    __syncthreads();
    const int lanes = n_shots <= kSelThreads / 16 ? 16 : 8, i = tid / lanes;
    const int sum = sum_of_no_lower(s_key, n_shots, i, tid % lanes, lanes);
    if (tid % lanes == 0 && i < n_shots) {
      if (prefix) s_keep[i] = sum <= shot_budget;
      else s_idx[sum - 1] = static_cast<uint16_t>(i);
    }
    __syncthreads();  // (also: the words' memory is free)
  } else if (prefix) {
    int len[kMaxPerThread];
    bool keep[kMaxPerThread];
#pragma unroll
    for (int j = 0; j < kMaxPerThread; ++j) {
      const int i = tid + kSelThreads * j;
      len[j] = i < n_shots ? s_off[i + 1] - s_off[i] : 0;
    }
    keep_prefix(my_score, len, n_shots, shot_budget, s_key, keep);
#pragma unroll
    for (int j = 0; j < kMaxPerThread; ++j) {
      const int i = tid + kSelThreads * j;
      if (i < n_shots) s_keep[i] = keep[j];
    }
    __syncthreads();  // (also: the histograms' memory becomes the scan array)
  } else {
    // ---- rank: sort one key per shot, descending --------------------------------------------------
    int n_pad = kMinPad;
    while (n_pad < n_shots) n_pad <<= 1;
    {
      uint64_t key[kMaxPerThread];
#pragma unroll
      for (int j = 0; j < kMaxPerThread; ++j) {
        const int i = tid + kSelThreads * j;
        key[j] = i < n_shots ? rank_key(my_score[j], i) : padding_key(i);
      }
      if (n_pad <= kSelThreads) {
        uint64_t k1[1] = {key[0]};
        sort_keys_descending<1>(k1, n_pad, s_key);
        key[0] = k1[0];
      } else if (n_pad <= 2 * kSelThreads) {
        uint64_t k2[2] = {key[0], key[1]};
        sort_keys_descending<2>(k2, n_pad, s_key);
        key[0] = k2[0];
        key[1] = k2[1];
      } else {
        sort_keys_descending<kMaxPerThread>(key, n_pad, s_key);
      }
#pragma unroll
      for (int j = 0; j < kMaxPerThread; ++j) {
        const int r = tid + kSelThreads * j;  // rank
        if (r < n_shots) s_idx[r] = static_cast<uint16_t>(0xFFFFFFFFu - static_cast<uint32_t>(key[j]));
      }
    }
    __syncthreads();  // the ranking is complete, and the exchange buffer is free to hold the lengths
  }
  if (!prefix) {
    // ---- budget walk in rank order -----------------------------------------------------------------
    for (int i = tid; i < n_shots; i += kSelThreads) {
      const int shot = s_idx[i];
      s_a[i] = s_off[shot + 1] - s_off[shot];
      s_keep[i] = 0;
    }
    __syncthreads();
    if (tid < kWave) first_fit_walk(s_a, s_idx, n_shots, shot_budget, s_keep);
    __syncthreads();
  }

  // ---- copy plan in position order: segment 0 = prefix, 1..n = shots, n+1 = tail ----------------
  // A segment's first output row and, among the segments that keep tokens, its number.
  const int n_seg = n_shots + 2;
  auto segment_start = [&](int s) { return s == 0 ? 0 : s_off[s - 1]; };
  auto segment_len = [&](int s) {
    if (s > 0 && s <= n_shots && !s_keep[s - 1]) return 0;
    return (s <= n_shots ? s_off[s] : n_tokens) - segment_start(s);
  };
  const int per = (n_seg + kSelThreads - 1) / kSelThreads, seg0 = min(tid * per, n_seg), seg1 = min(seg0 + per, n_seg);
  int row = 0, number = 0, total, n_kept;
  for (int s = seg0; s < seg1; ++s) {
    const int len = segment_len(s);
    row += len;
    number += len > 0;
  }
  block_exclusive_scan(row, number, total, n_kept, s_tmp);
  for (int s = seg0; s < seg1; ++s) {
    const int len = segment_len(s);
    if (len > 0) {
      s_a[number] = row;
      s_idx[number] = static_cast<uint16_t>(s);
      row += len;
      ++number;
    }
  }
  if (tid == 0) s_a[n_kept] = total;
  __syncthreads();
  // Every retained row's original position: a group of lanes per segment that keeps tokens, lanes along the rows; the
  // group is as wide as an average shot is long (a wave for shots of hundreds of tokens, 8..32 lanes for
  // sentence-sized units), so that most lanes have a row to write.
  int group_w = 8;
  {
    const int avg = n_shots > 0 ? (s_off[n_shots] - s_off[0]) / n_shots : kWave;
    while (group_w < kWave && group_w < avg) group_w <<= 1;
  }
  const int n_groups = kSelThreads / group_w, gid = tid / group_w, gl = tid % group_w;
  constexpr int kSegBatch = 4;  // segments whose LDS lookups are in flight together
  for (int k0 = gid; writes && k0 < n_kept; k0 += n_groups * kSegBatch) {
    int src[kSegBatch], len[kSegBatch], dst[kSegBatch];
#pragma unroll
    for (int b = 0; b < kSegBatch; ++b) {
      const int k = min(k0 + b * n_groups, n_kept - 1);
      dst[b] = s_a[k];
      len[b] = k0 + b * n_groups < n_kept ? s_a[k + 1] - dst[b] : 0;
      src[b] = segment_start(s_idx[k]);
    }
#pragma unroll
    for (int b = 0; b < kSegBatch; ++b)
      for (int i = gl; i < len[b]; i += group_w) kept_pos[dst[b] + i] = src[b] + i;
  }
  if (sel && writes) for (int i = tid; i < n_shots; i += kSelThreads) sel[i] = s_keep[i];
  if (tid == 0 && writes) { status[p] = SHOTKV_ST_OK; kept_count[p] = total; }

  // ---- this workgroup's share of the retained rows, of all planes ---------------------------------
  if constexpr (ROW_BYTES > 0) {
    constexpr int kLanes = ROW_BYTES / 16, kTeams = kSelThreads / kLanes;
    constexpr int kInFlight = 4;
    int* s_src = s_a + SHOTKV_MAX_SHOTS + 8;  // tokens of the share's rows
    static_assert(sizeof(uint64_t) * kKeySlots >= sizeof(int) * (SHOTKV_MAX_SHOTS + 8 + kSelThreads), "a share's rows fit");
    const int share_rows = ceil_div(total, static_cast<int>(gridDim.x)), row0 = blockIdx.x * share_rows;
    const int n_rows = min(share_rows, total - row0);  // at most one per thread
    if (n_rows <= 0) return;
    if (tid < n_rows) {
      int lo = 0, hi = n_kept;  // the segment that the row lies in: s_a[lo] <= row < s_a[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (s_a[mid] <= row0 + tid) lo = mid;
        else hi = mid;
      }
      s_src[tid] = segment_start(s_idx[lo]) + row0 + tid - s_a[lo];
    }
    __syncthreads();
    const int lane16 = 16 * (tid % kLanes), n_items = n_rows * 2 * H_kv;  // an item is a row of a plane
    const size_t plane0 = static_cast<size_t>(p) * H_kv;
    for (int t0 = tid / kLanes; t0 < n_items; t0 += kTeams * kInFlight) {
      u32x4 data[kInFlight];
      char* dst[kInFlight];
#pragma unroll
      for (int j = 0; j < kInFlight; ++j) {
        const int t = min(t0 + j * kTeams, n_items - 1), plane = t / n_rows, i = t - plane * n_rows;
        const bool is_v = plane >= H_kv;
        const size_t at = plane0 + (is_v ? plane - H_kv : plane);
        const char* src = (is_v ? copy.v : copy.k) + (at * n_tokens + s_src[i]) * ROW_BYTES + lane16;
        dst[j] = (is_v ? copy.v_out : copy.k_out) + (at * cap + row0 + i) * ROW_BYTES + lane16;
        data[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src));
      }
#pragma unroll
      for (int j = 0; j < kInFlight; ++j)
        if (t0 + j * kTeams < n_items) __builtin_nontemporal_store(data[j], reinterpret_cast<u32x4*>(dst[j]));
    }
  }
}

}  // namespace

hipError_t launch_reduce_select(const PrefillDims& d, bool with_mass, bool with_select, float* shot_scores,
                                const int32_t* shot_offsets, const int32_t* budget_tokens, int cap,
                                int32_t* kept_count, uint8_t* shot_selected, int32_t* status,
                                int32_t* kept_positions, const PrefillWorkspace& w, hipStream_t s) {
  KernelTimer timer(d.timing, kKernelReduceSelect, s);
  const int group_shift = 31 - __builtin_clz(static_cast<unsigned>(w.group_keys));
#define SHOTKV_LAUNCH_RS(M, S, RB, WGS, COPY)                                                           \
  hipLaunchKernelGGL((reduce_select_kernel<M, S, RB>), dim3(WGS, d.P), dim3(kSelThreads), 0, s, w.chunk_mass, \
                     w.max_c, group_shift, d.H_kv, shot_scores,                                         \
                     shot_offsets, budget_tokens, d.share, d.n_shots, d.n_tokens, cap, d.select_mode,   \
                     kept_count, shot_selected, status, kept_positions, COPY)
  if (with_mass && with_select) SHOTKV_LAUNCH_RS(true, true, 0, 1, CopyArgs{});
  else if (with_mass) SHOTKV_LAUNCH_RS(true, false, 0, 1, CopyArgs{});
  else if (with_select) SHOTKV_LAUNCH_RS(false, true, 0, 1, CopyArgs{});
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_select_compact(const PrefillDims& d, bool with_mass, float* shot_scores, const int32_t* shot_offsets,
                                 const int32_t* budget_tokens, const void* k, const void* v, void* k_out, void* v_out,
                                 int cap, int32_t* kept_count, uint8_t* shot_selected, int32_t* status,
                                 int32_t* kept_positions, const PrefillWorkspace& w, hipStream_t s) {
  const int row_bytes = d.D * (d.dtype == SHOTKV_BF16 ? 2 : 4);
  // Few rows: one launch, up to a workgroup per CU, each making the selection for itself and copying its share of the rows.
  // It saves a launch and the way of the positions through memory, but copies of many rows want many small workgroups and
  // the second workgroup of a CU slows the selections of both.  Whole calls, two launches and one, 8 KV heads, head_dim 128
  // unless told otherwise, by bytes read and written: 7 MB (2000 tokens) 23 and 20.5 us, 10 MB 22 and 20.6, 27 MB (8192
  // tokens, budget 3276) 25.6 and 23.7, with 128 workgroups 26.2, with 512 29; 54 MB 32.7 and 31.4; 33 MB as 64 problems
  // 28.6 and 27.5; 2500 units 77 and 75; 64 MB 130 and 130.5 (600 units), 79 MB of fp32 54.6 and 54.5, 210 MB of head_dim 64
  // 112 and 116, 322 MB 150 and 157.  That every workgroup sorts for first fit costs nothing either: one problem of 4000 units
  // 121.4 and 119.1, 2500 112.9 and 110.8, 8 of 1000 102.6 and 92.9, 64 of 600 102.2 and 100.5, 256 of 1000 198.6 and 198.8.
  constexpr int kMostWorkgroups = 256;
  const int most_rows = min(cap, d.n_tokens), wgs = max(1, min(kMostWorkgroups / d.P, ceil_div(cap, 8)));
  const long bytes = 4L * d.P * d.H_kv * most_rows * row_bytes;  // read and written
  if (bytes > 48L << 20 || d.P > kMostWorkgroups || ceil_div(most_rows, wgs) > kSelThreads) {
    const hipError_t e = launch_reduce_select(d, with_mass, true, shot_scores, shot_offsets, budget_tokens, cap, kept_count,
                                              shot_selected, status, kept_positions, w, s);
    return e != hipSuccess ? e : launch_compact(d, k, v, k_out, v_out, cap, kept_positions, kept_count, s);
  }
  { KernelTimer copy_timer(d.timing, kKernelCompact, s); }  // the copies are part of the same kernel
  KernelTimer timer(d.timing, kKernelReduceSelect, s);
  const int group_shift = 31 - __builtin_clz(static_cast<unsigned>(w.group_keys));
  const CopyArgs copy = {static_cast<const char*>(k), static_cast<const char*>(v), static_cast<char*>(k_out),
                         static_cast<char*>(v_out)};
#define SHOTKV_LAUNCH_SC(RB)                                                 \
  if (with_mass) SHOTKV_LAUNCH_RS(true, true, RB, wgs, copy);                \
  else SHOTKV_LAUNCH_RS(false, true, RB, wgs, copy)
  switch (row_bytes) {
    case 128: SHOTKV_LAUNCH_SC(128); break;
    case 256: SHOTKV_LAUNCH_SC(256); break;
    case 512: SHOTKV_LAUNCH_SC(512); break;
    default: return hipErrorInvalidValue;
  }
#undef SHOTKV_LAUNCH_SC
#undef SHOTKV_LAUNCH_RS
  return hipGetLastError();
}

}  // namespace shotkv
