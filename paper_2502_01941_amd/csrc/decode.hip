// Decode step over the compressed cache (Section 5.1, Eq. 7-9; Algorithm 1 phase 2).
//
// decode_partial : split-KV attention of the new query heads over [prefill rows | decode slots]
//                  (decode_mfma.hip): appends k_new/v_new to the lowest free slot, leaves every token
//                  range's softmax statistics and weighted value sum, and the scaled logits of the decode tokens.
// decode_finish  : per sequence, one workgroup computes Score(t) = sum_h alpha_{t,h} for the decode
//                  tokens (Eq. 7) and evicts the lowest-scored earlier token when the decode cache
//                  exceeds its budget (Eq. 8 in capacity form), while further workgroups merge the
//                  splits of four query heads each into the attention output.  (A kernel boundary
//                  after decode_partial is cheaper than a device-scope fence: the workgroups of a
//                  sequence sit on different XCDs with separate L2 caches.)
#include "common.hpp"

namespace shotkv {

namespace {

constexpr int kFinThreads = 1024;
constexpr int kFinWaves = kFinThreads / kWave;
constexpr int kFinMaxHeads = 64;

// lower score first, then the newer token: the order in which decode tokens are evicted
__device__ __forceinline__ bool evict_before(float sa, int pa, float sb, int pb) {
  return (sa < sb) | ((sa == sb) & (pa > pb));
}

// Of two eviction candidates the better one goes to (score, pos, slot); a slot of -1 is none.
__device__ __forceinline__ void take_better(float& score, int& pos, int& slot, float s, int p, int l) {
  const bool better = (l >= 0) & ((slot < 0) | evict_before(s, p, score, pos));
  score = better ? s : score;
  pos = better ? p : pos;
  slot = better ? l : slot;
}
template <int MASK>
__device__ __forceinline__ void take_better_of_lane(float& score, int& pos, int& slot) {
  take_better(score, pos, slot, __uint_as_float(lane_xor<MASK>(__float_as_uint(score))),
              static_cast<int>(lane_xor<MASK>(static_cast<uint32_t>(pos))),
              static_cast<int>(lane_xor<MASK>(static_cast<uint32_t>(slot))));
}

// Second half of a decode step.  Per sequence, workgroup 0 turns the decode-slot logits into
// Score(t) = sum over heads of the attention weight (Eq. 7) and retains under the budget (Eq. 8: the
// new token is exempt, the lowest score goes, the newest among equals); workgroups 1.. each merge the
// split partials of kFinHeadsPerGroup query heads into the attention output (Eq. 9).  Every workgroup
// first derives the softmax statistics of the heads it needs from the split partials.  The kernel is bound by
// its trips to memory, so what the second phase needs - the logits of the first round of slots, the first
// partials - is requested along with the first splits' statistics and all of it is one trip.  Those come first:
// loads return in order, and the statistics are worked out while 64 KB of logits follow.  Reductions stay off the
// LDS pipe.  One sequence of 3790 rows and 32 heads, whole step: 18.6 us with the statistics last and exchanges
// through LDS, 17.3 like this (kernel 7.8 and 7.1); 32 sequences of 2514 rows per KV head 41.0 and 39.5, 16 of
// 5121 67.4 and 66.5.
// kAhead: heads whose logits of a thread's first slot are requested that way.  32 cost 100 registers, one workgroup
// per CU, which is dear where heads are few and sequences many (per-KV-head mode: 256 pairs of 4 heads 12.1 us),
// so up to 8 heads take the small form.
constexpr int kFinHeadsPerGroup = 4;
// WHOLE: the outputs are written and z_dec holds H = H_kv partial scores per slot, to be added; only workgroup 0 is left.
template <int D, int kAhead, bool WHOLE>
__global__ __launch_bounds__(kFinThreads) void decode_finish_kernel(
    const float2* __restrict__ part_ml, const float* __restrict__ part_o,
    const float* __restrict__ z_dec, int32_t* __restrict__ slot_pos,
    const int32_t* __restrict__ new_slot_in, int n_slots, int H, int n_splits, int budget,
    int step_index, float* __restrict__ out, float* __restrict__ token_scores,
    int32_t* __restrict__ evicted_pos, int32_t* __restrict__ status) {
  const int s = blockIdx.y, tid = threadIdx.x;
  const int lane = tid % kWave, wave = tid / kWave;
  __shared__ float2 s_stat[kFinMaxHeads];  // per head: maximum, 1 / sum
  __shared__ float s_w[kFinHeadsPerGroup][kDecodeMaxSplits];  // merge workgroups only
  __shared__ __attribute__((aligned(16))) float s_o[kFinThreads * 4];  // merge workgroups only
  __shared__ float s_best_score[kFinWaves];
  __shared__ int s_best_pos[kFinWaves];
  __shared__ int s_best_slot[kFinWaves];
  __shared__ int s_count[kFinWaves];

  int32_t* sp = slot_pos + static_cast<size_t>(s) * n_slots;
  const int new_slot = new_slot_in[s];
  const size_t head0 = static_cast<size_t>(s) * H;
  const bool retain = WHOLE || blockIdx.x == 0;
  // heads whose statistics this workgroup needs: all of them for the scores, its own for the merge
  const int h_lo = retain ? 0 : (static_cast<int>(blockIdx.x) - 1) * kFinHeadsPerGroup;
  const int h_hi = retain ? H : min(h_lo + kFinHeadsPerGroup, H);

  // A pool of budget + 1 slots is one more than a round of threads: the few slots past the last full
  // round are scored by one wave each, lanes over the heads.
  constexpr int kMaxExtra = 4;  // per wave
  int n_extra = n_slots > kFinThreads ? n_slots % kFinThreads : 0;
  if (n_extra > kMaxExtra * kFinWaves) n_extra = 0;
  const int n_main = n_slots - n_extra;

  // ---- the first splits' statistics of a wave's first two heads: loads return in order, so they come first ----
  float m_first[2], l_first[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int h = h_lo + wave + i * kFinWaves;
    m_first[i] = -INFINITY;
    l_first[i] = 0.f;
    if (!WHOLE && h < h_hi && lane < n_splits) {
      const float2 ml = part_ml[(head0 + h) * n_splits + lane];
      m_first[i] = ml.x;
      l_first[i] = ml.y;
    }
  }

  // ---- what the second phase reads first -------------------------------------------------------------
  float z_first[kAhead];  // (a slot of no token may hold anything)
  int pos_first = -1;
  float ez[kMaxExtra];
  int epos[kMaxExtra];
  // merge: a thread takes four columns of one head and every kTeams-th split
  constexpr int kColumns = D / 4;
  constexpr int kTeams = kFinThreads / (kFinHeadsPerGroup * kColumns);
  const int mh = h_lo + tid / kColumns % kFinHeadsPerGroup, column = tid % kColumns;
  const int team = tid / (kColumns * kFinHeadsPerGroup);
  const float4* po = reinterpret_cast<const float4*>(part_o) + (head0 + min(mh, H - 1)) * n_splits * kColumns + column;
  constexpr int kPartsAhead = 4;
  float4 part_first[kPartsAhead];
  if (retain) {
#pragma unroll
    for (int h = 0; h < kAhead; ++h)
      z_first[h] = (h < H && tid < n_main) ? z_dec[(head0 + h) * n_slots + tid] : 0.f;
    if (tid < n_main) pos_first = sp[tid];
#pragma unroll
    for (int k = 0; k < kMaxExtra; ++k) {
      const int slot = n_main + wave + k * kFinWaves;
      ez[k] = -INFINITY;
      epos[k] = -1;
      if (slot < n_slots) {
        epos[k] = sp[slot];
        if (lane < H) ez[k] = z_dec[(head0 + lane) * n_slots + slot];
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < kPartsAhead; ++j) {
      const int i = team + j * kTeams;
      part_first[j] = i < n_splits ? po[static_cast<size_t>(i) * kColumns] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }

  // ---- global softmax statistics per head: one wave per head, lanes over the splits; each split's weight
  // 2^(m - M) is kept so that the merge below is a plain weighted sum
  // (a wave's heads are taken two at a time so that their first loads travel together)
  for (int h = h_lo + wave; !WHOLE && h < h_hi; h += 2 * kFinWaves) {
    const int h2 = h + kFinWaves;
    const bool two = h2 < h_hi;
    const float2* ml = part_ml + (head0 + h) * n_splits;
    const float2* ml2 = part_ml + (head0 + (two ? h2 : h)) * n_splits;
    // the first 64 splits stay in registers, any others are looked at twice (out of cache)
    const bool ahead = h < h_lo + 2 * kFinWaves;
    float m = m_first[0], l = l_first[0], m2 = m_first[1], l2 = l_first[1];
    if (!ahead) {
      m = m2 = -INFINITY;
      l = l2 = 0.f;
      if (lane < n_splits) { m = ml[lane].x; l = ml[lane].y; }
      if (lane < n_splits && two) { m2 = ml2[lane].x; l2 = ml2[lane].y; }
    }
    float M = m, M2 = m2;
    for (int i = lane + kWave; i < n_splits; i += kWave) {
      M = fmaxf(M, ml[i].x);
      M2 = fmaxf(M2, ml2[i].x);
    }
    M = wave_max(M);
    M2 = wave_max(M2);
    float L = 0.f, L2 = 0.f;
    auto add_split = [&](int i, float m, float l, float m2, float l2) {
      const float wgt = l > 0.f ? __builtin_amdgcn_exp2f(m - M) : 0.f;
      const float wgt2 = l2 > 0.f ? __builtin_amdgcn_exp2f(m2 - M2) : 0.f;
      L += l * wgt;
      L2 += l2 * wgt2;
      if (!retain) {
        s_w[h - h_lo][i] = wgt;
        if (two) s_w[h2 - h_lo][i] = wgt2;
      }
    };
    if (lane < n_splits) add_split(lane, m, l, m2, l2);
    for (int i = lane + kWave; i < n_splits; i += kWave) add_split(i, ml[i].x, ml[i].y, ml2[i].x, ml2[i].y);
    L = wave_sum(L);
    L2 = wave_sum(L2);
    if (lane == 0) {
      s_stat[h] = make_float2(M, 1.f / L);
      if (two) s_stat[h2] = make_float2(M2, 1.f / L2);
    }
  }
  if (new_slot < 0) {  // pool full: the step is void for this sequence
    if (retain) {
      if (token_scores)
        for (int i = tid; i < n_slots; i += kFinThreads) token_scores[static_cast<size_t>(s) * n_slots + i] = 0.f;
      if (tid == 0) {
        status[s] = SHOTKV_ST_NO_FREE_SLOT;
        if (evicted_pos) evicted_pos[s] = -1;
      }
    } else {
      for (int i = h_lo * D + tid; i < h_hi * D; i += kFinThreads) out[head0 * D + i] = 0.f;
    }
    return;
  }

  if (!WHOLE) __syncthreads();

  if (!retain) {  // attention output of this workgroup's heads
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    auto add = [&](const float4& x, float w) {
      acc.x = fmaf(x.x, w, acc.x);
      acc.y = fmaf(x.y, w, acc.y);
      acc.z = fmaf(x.z, w, acc.z);
      acc.w = fmaf(x.w, w, acc.w);
    };
    if (mh < h_hi) {
#pragma unroll
      for (int j = 0; j < kPartsAhead; ++j) {
        const int i = team + j * kTeams;
        if (i < n_splits) add(part_first[j], s_w[mh - h_lo][i]);
      }
      for (int i = team + kPartsAhead * kTeams; i < n_splits; i += kTeams)
        add(po[static_cast<size_t>(i) * kColumns], s_w[mh - h_lo][i]);
    }
    *reinterpret_cast<float4*>(&s_o[4 * tid]) = acc;
    __syncthreads();
    const int idx = h_lo * D + tid;  // team t's sums of these heads start at t * kFinHeadsPerGroup * D
    if (tid < kFinHeadsPerGroup * D && idx < h_hi * D) {
      float sum = 0.f;
#pragma unroll
      for (int t = 0; t < kTeams; ++t) sum += s_o[t * kFinHeadsPerGroup * D + tid];
      out[head0 * D + idx] = sum * s_stat[idx / D].y;
    }
    return;
  }

  // retention scores and the eviction candidate
  float best_score = INFINITY;
  int best_pos = -1, best_slot = -1, count = 0;
  auto share = [&](float z, int h) { return WHOLE ? z : __builtin_amdgcn_exp2f(z - s_stat[h].x) * s_stat[h].y; };
  constexpr int kHeadBatch = 16;  // loads in flight
  for (int slot = tid; slot < n_main; slot += kFinThreads) {
    const bool first = slot == tid;
    const int pos = (slot == new_slot) ? step_index : first ? pos_first : sp[slot];
    float score = 0.f;
    if (pos >= 0) {
      ++count;
      const float* z = z_dec + head0 * n_slots + slot;
      if (first) {
#pragma unroll
        for (int h = 0; h < kAhead; ++h)
          if (h < H) score += share(z_first[h], h);
      }
      for (int h0 = first ? kAhead : 0; h0 < H; h0 += kHeadBatch) {
        float zz[kHeadBatch];
#pragma unroll
        for (int j = 0; j < kHeadBatch; ++j) zz[j] = z[static_cast<size_t>(min(h0 + j, H - 1)) * n_slots];
#pragma unroll
        for (int j = 0; j < kHeadBatch; ++j)
          if (h0 + j < H) score += share(zz[j], h0 + j);
      }
      if (slot != new_slot) take_better(best_score, best_pos, best_slot, score, pos, slot);
    }
    if (token_scores) token_scores[static_cast<size_t>(s) * n_slots + slot] = score;
  }
#pragma unroll
  for (int k = 0; k < kMaxExtra; ++k) {
    const int slot = n_main + wave + k * kFinWaves;
    if (slot < n_slots) {  // wave-uniform
      const int pos = slot == new_slot ? step_index : epos[k];
      float part = 0.f;
      if (pos >= 0 && lane < H) part = share(ez[k], lane);
      // same order of the head sum as in the main loop would need a serial add; a tree sum over the
      // heads differs from it only in rounding, within the score tolerance
      const float score = wave_sum(part);
      if (lane == 0) {
        if (pos >= 0) {
          ++count;
          if (slot != new_slot) take_better(best_score, best_pos, best_slot, score, pos, slot);
        }
        if (token_scores) token_scores[static_cast<size_t>(s) * n_slots + slot] = score;
      }
    }
  }
  take_better_of_lane<32>(best_score, best_pos, best_slot);
  take_better_of_lane<16>(best_score, best_pos, best_slot);
  take_better_of_lane<8>(best_score, best_pos, best_slot);
  take_better_of_lane<4>(best_score, best_pos, best_slot);
  take_better_of_lane<2>(best_score, best_pos, best_slot);
  take_better_of_lane<1>(best_score, best_pos, best_slot);
  count = wave_sum(count);
  if (lane == 0) {
    s_best_score[wave] = best_score; s_best_pos[wave] = best_pos; s_best_slot[wave] = best_slot;
    s_count[wave] = count;
  }
  __syncthreads();  // also: every thread has read its slot_pos entries before thread 0 rewrites two
  if (wave == 0) {
    static_assert(kFinWaves == 16, "one row of lanes");
    best_score = s_best_score[lane % kFinWaves];
    best_pos = s_best_pos[lane % kFinWaves];
    best_slot = s_best_slot[lane % kFinWaves];
    const int total = wave_sum(lane < kFinWaves ? s_count[lane] : 0);
    take_better_of_lane<8>(best_score, best_pos, best_slot);
    take_better_of_lane<4>(best_score, best_pos, best_slot);
    take_better_of_lane<2>(best_score, best_pos, best_slot);
    take_better_of_lane<1>(best_score, best_pos, best_slot);
    if (lane == 0) {
      sp[new_slot] = step_index;
      int ev = -1;
      if (total > budget && best_slot >= 0) {
        ev = best_pos;
        sp[best_slot] = -1;
      }
      if (evicted_pos) evicted_pos[s] = ev;
      status[s] = SHOTKV_ST_OK;
    }
  }
}

}  // namespace

int decode_resident(int G, int row_bytes) { return G > 4 && row_bytes <= 256 ? 768 : 1024; }

int decode_splits(int S, int H_kv, int G, int row_bytes, int total_tokens) {
  // Token ranges per (sequence, KV head).  The workgroups of a launch should all be resident at once, so a count is rounded
  // down.  Whole steps, us, 8 KV heads, rows + slots of a sequence, head_dim 128 bf16 unless told otherwise.
  // With more than two query heads per KV head three workgroups per CU are better than four: 4 heads, 16 sequences of 4096 +
  // 1025 rows 64.0 with 768 workgroups and 65.7 with 1024, 24 of 3000 + 301 57.3 and 59.4 (960), of head_dim 64 34.7 and 37.0;
  // 12 of 4096 + 1025 51.8 and 51.0 (960).  One or two heads go either way: 2 heads, 24 of 3000 + 301 53.7 and 56.2, 33 of
  // 1800 + 101 49.2 (528) and 48.5 (792), one of head_dim 64, 16 of 4096 + 1025 33.6 and 32.4, 50 of 900 + 65 26.1 (400) and
  // 21.8 (800).  768 is passed over where it cannot be met within a sixth (4 heads, 33 of 1800 + 101 54.1 with 528 and 53.5 with
  // 792, of head_dim 64 32.8 and 31.4; 64 of 300 + 65 29.8 and 29.4; 20 of 2000 + 301 38.9 with 640 and 39.7 with 960) - but not
  // with more than four heads of up to 256 bytes: bf16 rows leave room for three per CU (137 registers), 8 heads, 33 of 1800 +
  // 101, 67.0 with 528 and 73.6 with 792, 50 of 900 + 65 62.1 with 400 and 66.2 with 800, 5 heads 57.7 and 60.2.  fp32 rows
  // leave room for four, and gain by it with 512 bytes (50 of 900 + 65: 102.7 and 94.6); with 256 bytes they would too (78.2
  // and 72.6, 70.4 and 62.5), but steps that the static scratch memory holds would then outgrow it.
  const int pairs = S * H_kv;
  const int many = max(1, decode_resident(G, row_bytes) / pairs), few = max(1, 768 / pairs);
  int splits = G > 2 && few * pairs >= 640 ? few : many;
  // no range shorter than 96 tokens, or 64 where that makes no more than two workgroups per CU (one sequence of 3800 rows,
  // 8 KV heads: 17.0 us with 96, 16.8 with 64, 18.4 with 128; of 1100 rows, 4 KV heads, 17.8, 15.4 and 17.8; 8 sequences
  // of 600 fp32 rows 19.1, 19.5 and 20.9) ...
  splits = min(splits, max(1, total_tokens / (pairs * (total_tokens / 64) <= 512 ? 64 : 96)));
  // ... none longer than one piece of logits per workgroup, and no more than the finish kernel takes
  splits = max(splits, ceil_div(total_tokens, kDecodeMaxRange));
  return max(1, min(splits, kDecodeMaxSplits));
}

// Whether one workgroup takes all tokens of a (sequence, KV head).  It knows the whole softmax, so it writes the output
// and one partial score per slot instead of partial sums of every range and the logits of every head: those writes, a
// hundredth of the bytes read, cost the row stream an eighth of its time (512 sequences of 5121 rows, 8 KV heads: step
// 1840 us, 1760 without storing logits, 1600 without partial sums either, 1640 like this, where the finish kernel shrinks
// from 51 to 12 as well).  But a workgroup takes as long as its sequence, and a launch as long as its last workgroup, so it
// is for launches of rounds enough that both the lengths and the last round even out: two rounds of the three (three or four
// query heads per KV head), four (two) or two workgroups (seven or eight, and rows of 128 bytes) per CU that share the chip
// best, with three quarters of the rounds' places taken.  Whole steps, us, ranges and whole; rows in use 94 to 100 % of the
// capacity ("even"), uniform from 3 to 100 % of it, all in every other sequence and a quarter in the rest ("half"), all in
// every 16th and a sixteenth in the rest ("few long"); 8 KV heads, head_dim 128 bf16 unless told otherwise:
//   one round, 4 heads: 96 x 4096 + 512 even 308 and 268, uniform 213 and 206, half 239 and 213, few long 116 and 187; 64 x
//     4096 + 512 208 and 184, 148 and 164, 163 and 169, 83 and 160; fp32, 96 x 2000 + 64, 264 and 253, 180 and 186, 209 and
//     209, 87 and 172; 2 heads, head_dim 64, 128 x 2000 + 64, 96 and 102, 70 and 73, 78 and 88, 45 and 52
//   two rounds and more, 4 heads: 192 x 3163 + 64 even 421 and 386, uniform 308 and 258, few long 136 and 156; 256 562 and 520,
//     407 and 330, 175 and 186; 384 851 and 786, 618 and 493, 257 and 259; 576 1274 and 1171, 915 and 697, 376 and 352; 2
//     heads, 256 x 1200 + 64, 223 and 209, 158 and 139, 87 and 83; fp32, head_dim 64, 336 x 1500 + 100, 350 and 335, 243 and
//     218, half 256 and 262, few long 124 and 136
//   a third round begun: 200 x 1200 + 64 (69 % of three) even 185 and 194, fp32 346 and 365; 216 (75 %) 201 and 198, 375 and 375
//   one head gains too little: 288 x 1500 + 100 even 294 and 296, uniform 205 and 189, half 215 and 229, few long 97 and 104; 400
//     399 and 398, 271 and 248, 287 and 298, 126 and 135
//   5 to 8 heads, two workgroups per CU, head_dim 64: 8 heads, 4 KV heads, 256 x 1784 + 407 even 136 and 123, uniform 113 and
//     115, few long 93 and 108, 512 of them 256 and 241, 210 and 202, 167 and 185; 7 heads, 256 156 and 122, 133 and 114, 113
//     and 108; 5 heads, 256 129 and 122, 108 and 114, 88 and 107, of 8 KV heads, 192 x 1200 + 64, 118 and 126; head_dim 128, 8
//     heads, 2048 pairs of 1200 + 64, 278 and 283
// Where one range is all there is anyway nothing is won.
bool decode_whole(const DecodeDims& d, int row_bytes) {
  if (d.n_splits < 2 || d.n_slots > decode_map_rows(row_bytes)) return false;
  if (d.G == 1 || (d.G > 4 && (d.G < 7 || row_bytes > 128))) return false;
  const int round = d.G > 4 ? 512 : d.G > 2 ? 768 : 1024, pairs = d.S * d.H_kv;
  return pairs >= 2 * round && 4L * pairs >= 3L * round * ceil_div(pairs, round);
}

hipError_t launch_decode_finish(const DecodeDims& d, const shotkv_decode_state& st, float* out,
                                float* token_scores, int32_t* evicted_pos, int32_t* status,
                                const DecodeWorkspace& w, hipStream_t s) {
  if (d.H > kFinMaxHeads || d.n_splits > kDecodeMaxSplits) return hipErrorInvalidValue;
  KernelTimer timer(d.timing, kKernelDecodeFinish, s);
  const int rows = d.whole ? d.H_kv : d.H;
  const dim3 grid(d.whole ? 1 : 1 + ceil_div(d.H, kFinHeadsPerGroup), d.S);
  auto* kernel = d.whole       ? (rows <= 8 ? decode_finish_kernel<128, 8, true> : decode_finish_kernel<128, 32, true>)
                 : d.D == 128 ? (rows <= 8 ? decode_finish_kernel<128, 8, false> : decode_finish_kernel<128, 32, false>)
                              : (rows <= 8 ? decode_finish_kernel<64, 8, false> : decode_finish_kernel<64, 32, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(kFinThreads), 0, s, w.part_ml, w.part_o, w.z_dec, st.slot_pos, w.new_slot,
                     d.n_slots, rows, d.n_splits, d.budget, d.step, out, token_scores, evicted_pos, status);
  return hipGetLastError();
}

}  // namespace shotkv
