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
  return sa < sb || (sa == sb && pa > pb);
}

// Second half of a decode step.  Per sequence, workgroup 0 turns the decode-slot logits into
// Score(t) = sum over heads of the attention weight (Eq. 7) and retains under the budget (Eq. 8: the
// new token is exempt, the lowest score goes, the newest among equals); workgroups 1.. each merge the
// split partials of kFinHeadsPerGroup query heads into the attention output (Eq. 9).  Every workgroup
// first derives the softmax statistics of the heads it needs from the split partials; after that all
// of its loads are independent of one another, so the kernel costs two memory round trips.
constexpr int kFinHeadsPerGroup = 4;
__global__ __launch_bounds__(kFinThreads) void decode_finish_kernel(
    const float2* __restrict__ part_ml, const float* __restrict__ part_o,
    const float* __restrict__ z_dec, int32_t* __restrict__ slot_pos,
    const int32_t* __restrict__ new_slot_in, int n_slots, int H, int D, int n_splits, int budget,
    int step_index, float* __restrict__ out, float* __restrict__ token_scores,
    int32_t* __restrict__ evicted_pos, int32_t* __restrict__ status) {
  const int s = blockIdx.y, tid = threadIdx.x;
  const int lane = tid % kWave, wave = tid / kWave;
  __shared__ float s_M[kFinMaxHeads];
  __shared__ float s_invL[kFinMaxHeads];
  __shared__ float s_w[kFinHeadsPerGroup][kDecodeMaxSplits];  // merge workgroups only
  __shared__ float s_best_score[kFinWaves];
  __shared__ int s_best_pos[kFinWaves];
  __shared__ int s_best_slot[kFinWaves];
  __shared__ int s_count[kFinWaves];

  int32_t* sp = slot_pos + static_cast<size_t>(s) * n_slots;
  const int new_slot = new_slot_in[s];
  const size_t head0 = static_cast<size_t>(s) * H;
  const bool retain = blockIdx.x == 0;
  // heads whose statistics this workgroup needs: all of them for the scores, its own for the merge
  const int h_lo = retain ? 0 : (static_cast<int>(blockIdx.x) - 1) * kFinHeadsPerGroup;
  const int h_hi = retain ? H : min(h_lo + kFinHeadsPerGroup, H);
  // (requested before the slot index above is looked at, so that the two loads travel together)
  // global softmax statistics per head: one wave per head, lanes over the splits; each split's weight
  // 2^(m - M) is kept so that the merge below is a plain weighted sum
  // (a wave's heads are taken two at a time so that their first loads travel together)
  for (int h = h_lo + wave; h < h_hi; h += 2 * kFinWaves) {
    const int h2 = h + kFinWaves;
    const bool two = h2 < h_hi;
    const float2* ml = part_ml + (head0 + h) * n_splits;
    const float2* ml2 = part_ml + (head0 + (two ? h2 : h)) * n_splits;
    float M = -INFINITY, M2 = -INFINITY;
    for (int i = lane; i < n_splits; i += kWave) {
      const float a = ml[i].x, b = ml2[i].x;
      M = fmaxf(M, a);
      M2 = fmaxf(M2, b);
    }
    M = wave_max(M);
    M2 = wave_max(M2);
    float L = 0.f, L2 = 0.f;
    for (int i = lane; i < n_splits; i += kWave) {  // second look at the same few bytes: out of cache
      const float2 x = ml[i], y = ml2[i];
      const float wgt = x.y > 0.f ? __builtin_amdgcn_exp2f(x.x - M) : 0.f;
      const float wgt2 = y.y > 0.f ? __builtin_amdgcn_exp2f(y.x - M2) : 0.f;
      L += x.y * wgt;
      L2 += y.y * wgt2;
      if (!retain) {
        s_w[h - h_lo][i] = wgt;
        if (two) s_w[h2 - h_lo][i] = wgt2;
      }
    }
    L = wave_sum(L);
    L2 = wave_sum(L2);
    if (lane == 0) {
      s_M[h] = M; s_invL[h] = 1.f / L;
      if (two) { s_M[h2] = M2; s_invL[h2] = 1.f / L2; }
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

  __syncthreads();

  if (!retain) {  // attention output of this workgroup's heads
    for (int idx = h_lo * D + tid; idx < h_hi * D; idx += kFinThreads) {
      const int h = idx / D, dd = idx - h * D;
      const float* po = part_o + (head0 + h) * n_splits * D + dd;
      float acc = 0.f;
      for (int i = 0; i < n_splits; ++i) acc = fmaf(po[static_cast<size_t>(i) * D], s_w[h - h_lo][i], acc);
      out[(head0 + h) * D + dd] = acc * s_invL[h];
    }
    return;
  }

  // retention scores and the eviction candidate
  float best_score = INFINITY;
  int best_pos = -1, best_slot = -1, count = 0;
  // A pool of budget + 1 slots is one more than a round of threads: the few slots past the last full
  // round are scored by one wave each, lanes over the heads, and their logits are requested here, ahead
  // of the main loop, so that they do not cost a dependent trip to memory of their own.
  constexpr int kMaxExtra = 4;  // per wave
  int n_extra = n_slots > kFinThreads ? n_slots % kFinThreads : 0;
  if (n_extra > kMaxExtra * kFinWaves) n_extra = 0;
  const int n_main = n_slots - n_extra;
  float ez[kMaxExtra];
  int epos[kMaxExtra];
#pragma unroll
  for (int k = 0; k < kMaxExtra; ++k) {
    const int slot = n_main + wave + k * kFinWaves;
    ez[k] = -INFINITY;
    epos[k] = -1;
    if (slot < n_slots) {
      epos[k] = (slot == new_slot) ? step_index : sp[slot];
      if (lane < H) ez[k] = z_dec[(head0 + lane) * n_slots + slot];
    }
  }
  for (int slot = tid; slot < n_main; slot += kFinThreads) {
    const int pos = (slot == new_slot) ? step_index : sp[slot];
    float score = 0.f;
    if (pos >= 0) {
      ++count;
      const float* z = z_dec + head0 * n_slots + slot;
      for (int h = 0; h < H; ++h)
        score += __builtin_amdgcn_exp2f(z[static_cast<size_t>(h) * n_slots] - s_M[h]) * s_invL[h];
      if (slot != new_slot && (best_slot < 0 || evict_before(score, pos, best_score, best_pos))) {
        best_score = score; best_pos = pos; best_slot = slot;
      }
    }
    if (token_scores) token_scores[static_cast<size_t>(s) * n_slots + slot] = score;
  }
#pragma unroll
  for (int k = 0; k < kMaxExtra; ++k) {
    const int slot = n_main + wave + k * kFinWaves;
    if (slot < n_slots) {  // wave-uniform
      const int pos = epos[k];
      float part = 0.f;
      if (pos >= 0 && lane < H) part = __builtin_amdgcn_exp2f(ez[k] - s_M[lane]) * s_invL[lane];
      // same order of the head sum as in the main loop would need a serial add; a tree sum over the
      // heads differs from it only in rounding, within the score tolerance
      const float score = wave_sum(part);
      if (lane == 0) {
        if (pos >= 0) {
          ++count;
          if (slot != new_slot && (best_slot < 0 || evict_before(score, pos, best_score, best_pos))) {
            best_score = score; best_pos = pos; best_slot = slot;
          }
        }
        if (token_scores) token_scores[static_cast<size_t>(s) * n_slots + slot] = score;
      }
    }
  }
  for (int o = kWave / 2; o > 0; o >>= 1) {
    const float os = __shfl_xor(best_score, o, kWave);
    const int op = __shfl_xor(best_pos, o, kWave);
    const int ol = __shfl_xor(best_slot, o, kWave);
    count += __shfl_xor(count, o, kWave);
    if (ol >= 0 && (best_slot < 0 || evict_before(os, op, best_score, best_pos))) {
      best_score = os; best_pos = op; best_slot = ol;
    }
  }
  if (lane == 0) {
    s_best_score[wave] = best_score; s_best_pos[wave] = best_pos;
    s_best_slot[wave] = best_slot; s_count[wave] = count;
  }
  __syncthreads();  // also: every thread has read its slot_pos entries before thread 0 rewrites two
  if (tid == 0) {
    int total = s_count[0];  // this thread already holds wave 0's candidate
    for (int w = 1; w < kFinWaves; ++w) {
      total += s_count[w];
      if (s_best_slot[w] >= 0 &&
          (best_slot < 0 || evict_before(s_best_score[w], s_best_pos[w], best_score, best_pos))) {
        best_score = s_best_score[w]; best_pos = s_best_pos[w]; best_slot = s_best_slot[w];
      }
    }
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

}  // namespace

int decode_splits(int S, int H_kv, int G, int total_tokens) {
  // Token ranges per (sequence, KV head).  The workgroups of a launch should all be resident at once, so a count is
  // rounded down: 1056 workgroups of which 1024 fit take nearly twice as long as 960.  With more than two query
  // heads per KV head three workgroups per CU are better than four (and with more than four that is what fits):
  // 16 sequences of 4500 rows and 8 heads 73 us at 768 workgroups, 85 at 1024; 12 sequences of 5120 rows and 4
  // heads 55 and 58 (62 at 1056); 16 of 5120 rows 69.8 and 70.8.  One or two heads: 54.1 and 52.8 us at 16
  // sequences.  768 is passed over where it cannot be met within a sixth (64 sequences of 364 rows: 34.5 us with
  // 512 workgroups, 33.8 with 1024).
  const int pairs = S * H_kv;
  const int many = max(1, 1024 / pairs), few = max(1, 768 / pairs);
  int splits = G > 2 && few * pairs >= 640 ? few : many;
  // no range shorter than 96 tokens (one sequence of 3800 rows: 20.5 us, 21.6 with 128, 25 with 32) ...
  splits = min(splits, max(1, total_tokens / 96));
  // ... none longer than one piece of logits per workgroup, and no more than the finish kernel takes
  splits = max(splits, ceil_div(total_tokens, kDecodeMaxRange));
  return max(1, min(splits, kDecodeMaxSplits));
}

hipError_t launch_decode_finish(const DecodeDims& d, const shotkv_decode_state& st, float* out,
                                float* token_scores, int32_t* evicted_pos, int32_t* status,
                                const DecodeWorkspace& w, hipStream_t s) {
  if (d.H > kFinMaxHeads || d.n_splits > kDecodeMaxSplits) return hipErrorInvalidValue;
  KernelTimer timer(d.timing, kKernelDecodeFinish, s);
  hipLaunchKernelGGL(decode_finish_kernel, dim3(1 + ceil_div(d.H, kFinHeadsPerGroup), d.S), dim3(kFinThreads), 0, s, w.part_ml, w.part_o, w.z_dec,
                     st.slot_pos, w.new_slot, d.n_slots, d.H, d.D, d.n_splits, d.budget, d.step, out,
                     token_scores, evicted_pos, status);
  return hipGetLastError();
}

}  // namespace shotkv
